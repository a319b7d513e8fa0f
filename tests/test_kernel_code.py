"""The device code of the built library, read back as assembly: what the kernels rely on and the compiler does not
check.  The compute-bound kernels write their matrix products as inline assembly with the sums in the accumulation
registers, which hides them from the compiler's hazard pass (mfma16_acc in csrc/common.h); no kernel may spill."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2604_17709_amd as dn

LLVM = "/opt/rocm/llvm/bin"
TOOLS = {t: os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump", "llvm-readobj")}

# Wait states between a vector instruction that writes an operand or a sum of a matrix product and the product, and between a
# product of eight passes (16x16x32) and another use of its result.
OPERAND_WAIT, RESULT_WAIT = 2, 11

INSTRUCTION = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):")
REGISTER = re.compile(r"^\|?-?([va])(?:(\d+)|\[(\d+):(\d+)\])\|?$")


def registers(text):
    m = REGISTER.match(text.strip())
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {(m[1], i) for i in range(lo, hi + 1)}


def parse(lines):
    """[(address, opcode, operands, branch target or None)] of one kernel's listing."""
    out = []
    for line in lines:
        m = INSTRUCTION.match(line)
        if not m:
            continue
        target = None
        if m[1].startswith(("s_branch", "s_cbranch")):
            t = re.search(r"<[^>]*\+0x([0-9a-f]+)>", line)
            target = int(t[1], 16) if t else 0
        out.append((int(m[3], 16), m[1], m[2].split(", "), target))
    return out


def wait_states(op, operands):
    return int(operands[0], 0) + 1 if op == "s_nop" else 1


def paths_back(code):
    """For every instruction the indices it can be reached from: the one before it and the branches to it."""
    start = code[0][0]
    index = {c[0] - start: i for i, c in enumerate(code)}
    before = [[i - 1] if i and code[i - 1][1] not in ("s_branch", "s_endpgm") else [] for i in range(len(code))]
    for i, c in enumerate(code):
        if c[3] is not None and c[3] in index:
            before[index[c[3]]].append(i)
    return before


def hazards(lines):
    """The hazards around the products with sums in accumulation registers, as texts."""
    code = parse(lines)
    if not code:
        return 0, []
    before, found, products = paths_back(code), [], 0

    def walk(i, limit, visit, states=0):
        for j in before[i]:
            if visit(j):
                found.append("%x: %s %s after %x: %s %s" % (code[i0][0], code[i0][1], ", ".join(code[i0][2]), code[j][0], code[j][1], ", ".join(code[j][2])))
            n = states + wait_states(code[j][1], code[j][2])
            if n < limit:
                walk(j, limit, visit, n)

    for i0, (_, op, ops, _) in enumerate(code):
        if op.startswith("v_mfma") and ops[0].startswith("a"):
            products += 1
            need = registers(ops[1]) | registers(ops[2]) | registers(ops[3])
            walk(i0, OPERAND_WAIT, lambda j: code[j][1].startswith("v_") and not code[j][1].startswith(("v_mfma", "v_cmp", "v_readfirstlane", "v_readlane"))
                 and bool(registers(code[j][2][0]) & need))
        else:
            used = {r for o in ops for r in registers(o) if r[0] == "a"}
            if used:
                walk(i0, RESULT_WAIT, lambda j: code[j][1].startswith("v_mfma") and bool(registers(code[j][2][0]) & used))
    return products, found


@pytest.fixture(scope="module")
def device_code(tmp_path_factory):
    missing = [t for t in TOOLS.values() if not os.path.exists(t)]
    assert not missing, missing
    d = tmp_path_factory.mktemp("device_code")
    lib = str(d / "lib.so")
    shutil.copy(dn.LIB_PATH, lib)
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout
    run(TOOLS["llvm-objcopy"], "--dump-section=.hip_fatbin=%s" % (d / "fatbin"), lib)
    run(TOOLS["clang-offload-bundler"], "--unbundle", "--type=o", "--input=%s" % (d / "fatbin"),
        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=%s" % (d / "code"))
    return str(d / "code"), run


def test_no_kernel_spills(device_code):
    path, run = device_code
    notes = run(TOOLS["llvm-readobj"], "--notes", path)
    kernels = re.split(r"\n\s+- \.agpr_count:", notes)[1:]
    assert len(kernels) > 100
    for k in kernels:
        name = re.search(r"\.name:\s+(_Z\S+)", k)[1]
        for field in (r"\.private_segment_fixed_size", r"\.vgpr_spill_count", r"\.sgpr_spill_count"):
            assert int(re.search(field + r":\s+(\d+)", k)[1]) == 0, (name, field)


def test_products_on_accumulation_registers_have_no_hazard(device_code):
    path, _ = device_code
    proc = subprocess.Popen([TOOLS["llvm-objdump"], "-d", path], stdout=subprocess.PIPE, text=True)
    kernels = products = 0
    name, lines = "", []

    def check():
        nonlocal kernels, products
        if name and ("prefill" in name or "probe_mfma" in name):
            n, found = hazards(lines)
            assert not found, (name, found[:5])
            kernels, products = kernels + 1, products + n

    for line in proc.stdout:
        if line.endswith(">:\n"):
            check()
            name, lines = line, []
        elif "prefill" in name or "probe_mfma" in name:
            lines.append(line)
    check()
    assert proc.wait() == 0
    assert kernels >= 30 and products > 64 * kernels      # (every kernel has at least one stage of 64 products)


def listing(*code):
    return ["\t%s // %012X: 00000000" % (c, 4 * i) for i, c in enumerate(code)]


def test_the_hazard_check_finds_planted_hazards():
    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[0:3]"
    read = "v_accvgpr_read_b32 v0, a2"
    assert hazards(listing("ds_read_b128 v[8:11], v2", "s_nop 0", mfma)) == (1, [])
    for write in ("v_mov_b32_e32 v9, v1", "v_add_u32_e32 v15, 1, v3"):
        assert len(hazards(listing(write, mfma))[1]) == 1
        assert len(hazards(listing(write, "s_mov_b32 s0, 0", mfma))[1]) == 1
        assert hazards(listing(write, "s_nop 1", mfma))[1] == []
    assert hazards(listing("v_mov_b32_e32 v7, v1", mfma))[1] == []
    assert len(hazards(listing("v_accvgpr_write_b32 a1, 0", mfma))[1]) == 1
    assert len(hazards(listing(mfma, "s_nop 9", read))[1]) == 1
    assert hazards(listing(mfma, "s_nop 15", "s_nop 15", read))[1] == []
    # round a loop: the write at its end, the product at its start
    loop = listing(mfma, "s_nop 3", "v_mov_b32_e32 v8, v1", "s_cbranch_scc1 65532")
    loop[-1] += " <k+0x0>"
    assert len(hazards(loop)[1]) == 1
