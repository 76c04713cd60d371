"""The dense GEMM kernels issue their products as inline assembly, so the compiler does not know how long a result takes: if
it copied or spilled an accumulator inside the loop, it would read the register before the product has landed.  This compiles
the kernels as the library is built and checks in their assembly that it does not, and what they keep in scratch memory.  The
exchange of the column sums is inline assembly as well: its operands are checked the same way."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2506_03275_amd import build

# registers that may go to scratch memory, by kernel instance <form, rows of P>; all of it lies outside the product loops
SPILLS = {(0, 256): 0, (1, 256): 4, (2, 128): 0, (2, 256): 0, (3, 128): 0, (3, 192): 0}


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "mlp.s"
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "mlp.hip"), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


def _kernels(text):
    """{(form, rows of P): instruction and label lines}"""
    found = {}
    for m in re.finditer(r"^(_ZN\w*mlp_dense_gemm_kernelILi(\d+)ELi(\d+)E\w*):(.*?)^\s*\.size\s+\1,", text, re.S | re.M):
        lines = (line.split(";")[0].strip() for line in m[4].split("\n"))
        found[int(m[2]), int(m[3])] = [line for line in lines if line and not re.match(r"\.(?!L)", line)]
    return found


def _registers(operand_text, kind):
    regs = set()
    for first, last in re.findall(rf"(?<![\w]){kind}\[(\d+):(\d+)\]", operand_text):
        regs |= set(range(int(first), int(last) + 1))
    return regs | {int(r) for r in re.findall(rf"(?<![\w\[:]){kind}(\d+)\b", operand_text)}


def _is_product(line):
    return line.startswith("v_mfma")


def _faults(lines):
    """What would let a result be used before it has landed, or an operand before it is there."""
    products = [i for i, line in enumerate(lines) if _is_product(line)]
    accumulators = set().union(*(_registers(lines[i].split(",")[0], "a") for i in products))
    labels = {line[:-1]: i for i, line in enumerate(lines) if line.endswith(":")}
    loops = []
    for i, line in enumerate(lines):
        m = re.match(r"s_c?branch\w*\s+(\.L\w+)", line)
        if m and labels.get(m[1], i) < i:
            loops.append((labels[m[1]], i))
    with_products = [(a, b) for a, b in loops if any(a < i < b for i in products)]
    innermost = [(a, b) for a, b in with_products if not any(a < c and d <= b for c, d in with_products)]
    faults = []
    if not innermost or not all(any(a < i < b for a, b in innermost) for i in products):
        faults.append("a product outside the loops that were looked at")
    for a, b in innermost:
        faults += [f"in a loop: {line}" for line in lines[a:b] if not _is_product(line) and _registers(line, "a") & accumulators]
    for i in products:   # up to the wait that ends a loop's last products
        for j in range(i + 1, len(lines) - 1):
            if lines[j] == "s_nop 15" and lines[j + 1] == "s_nop 15":
                break
            if not _is_product(lines[j]) and _registers(lines[j], "a") & accumulators:
                faults.append(f"ahead of the wait: {lines[j]}")
                break
        else:
            faults.append("no wait behind a product")
        sources = _registers(lines[i].split(",", 1)[1], "v")
        for line in lines[i - 2:i]:   # two wait states between a vector write and a product that reads it
            if line.startswith("v_") and not _is_product(line) and _registers(line.split(",")[0], "v") & sources:
                faults.append(f"right ahead of a product that reads it: {line}")
    return faults


def test_no_accumulator_is_touched_before_its_product_has_landed(assembly):
    kernels = _kernels(assembly)
    assert set(kernels) == set(SPILLS)
    for form, lines in kernels.items():
        assert not _faults(lines), form


def test_the_check_sees_what_it_is_for(assembly):
    lines = _kernels(assembly)[0, 256]
    products = [i for i, line in enumerate(lines) if _is_product(line)]
    register = "a" + str(min(_registers(lines[products[0]].split(",")[0], "a")))
    copy = [f"v_accvgpr_read_b32 v0, {register}"]
    assert _faults(lines[:products[3]] + copy + lines[products[3]:])             # a copy between the products
    assert _faults(lines[:products[-1] + 1] + copy + lines[products[-1] + 1:])   # and ahead of the wait
    waits = [i for i, line in enumerate(lines) if line == "s_nop 15"]
    assert _faults([line for i, line in enumerate(lines) if i not in waits])     # no wait at all
    source = re.search(r"v\[(\d+):", lines[products[5]])[1]
    assert _faults(lines[:products[5]] + [f"v_mov_b32_e32 v{source}, 0"] + lines[products[5]:])


def test_registers_in_scratch_memory(assembly):
    spills = re.findall(r"\.name:\s+_ZN\w*mlp_dense_gemm_kernelILi(\d+)ELi(\d+)E.*?\.vgpr_spill_count:\s*(\d+)", assembly, re.S)
    assert {(int(form), int(rows)): int(n) for form, rows, n in spills} == SPILLS


def test_the_column_sums_exchange_keeps_its_inputs_apart(tmp_path):
    """The exchange writes its first four values before it has read the other four.  Called with the second four equal to the
    first, which the compiler sees, no input may share a register with what is written before it is read."""
    text = open(os.path.join(build.CSRC, "attn.hip")).read()
    start, end = text.index("template <int CTRL>\n"), text.index("// COLSUM (Alg. 4): also the tile's column sums")
    (tmp_path / "exchange.hip").write_text('#include "%s"\nnamespace chipmunk {\n%s\n}\nusing namespace chipmunk;\n'
        '__global__ void equal_halves(const float* in, float* out) {\n'
        '    __shared__ float part[32];\n    float x[8];\n'
        '    for (int i = 0; i < 4; i++) x[i] = x[i + 4] = in[threadIdx.x * 4 + i];\n'
        '    row16_sums_to_lds(x, part, threadIdx.x >> 4, threadIdx.x & 15);\n    __syncthreads();\n'
        '    out[threadIdx.x] = part[threadIdx.x & 31];\n}\n' % (os.path.join(build.CSRC, "common.h"), text[start:end]))
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-device-only", "-S",
                    str(tmp_path / "exchange.hip"), "-o", str(tmp_path / "exchange.s")], check=True, capture_output=True)
    adds = [[int(r) for r in re.findall(r"\bv(\d+)", line)] for line in (tmp_path / "exchange.s").read_text().split("\n")
            if re.match(r"\s*v_add_f32_dpp v\d+, v(\d+), v\1 row_(half_)?mirror\b", line)]
    assert len(adds) == 12
    written = {a[0] for a in adds[:4]}
    assert len(written) == 4 and all(a[0] == a[1] for a in adds[:4])
    assert not written & {a[1] for a in adds[4:8]}


def test_whole_rounds_of_narrow_heads_keep_their_workgroups(tmp_path):
    """The attention kernel holds the walk of whole chunks and that of the parts behind them.  For chunks of 128 rows at E = 64 the
    first fits 128 registers, four workgroups to a CU; no column list may be walked by an instance whose other walk takes
    more."""
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "attn.hip"), "-o", str(tmp_path / "attn.s")], check=True, capture_output=True)
    metadata = re.findall(r"\.name:\s+_ZN\w*attn_sparse_delta_kernelILi64ELi2ELi4ELi0ELi(\d)E.*?\.vgpr_count:\s*(\d+).*?"
                          r"\.vgpr_spill_count:\s*(\d+)", (tmp_path / "attn.s").read_text(), re.S)
    assert {int(part) for part, _, _ in metadata} == {0, 2}   # a workgroup per 64 rows, and per 32
    assert all(int(registers) <= 128 and spilled == "0" for _, registers, spilled in metadata), metadata
    form = ctypes.CDLL(build.LIB).chipmunk_internal_attn_part_form   # B, H, N, E, c, keys of a list (0: every column), list
    assert form(1, 11, 7500, 64, 128, 2500, 1) == 0 and form(1, 16, 7500, 64, 192, 2500, 1) == 1
