"""What the kernels' sources must hold to and no run shows: properties that hold or fail when the compiler allocates
registers and LDS."""
import glob
import os
import re
import subprocess

import pytest

from paper_2410_16926_amd import build

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_16926_amd", "csrc")
SOURCES = sorted(os.path.basename(p) for pattern in ("*.hip", "*.h") for p in glob.glob(os.path.join(CSRC, pattern)))

# a load whose result comes into registers (loads into LDS have none)
LOAD = re.compile(r"\b(ds_(read|load|bpermute|permute|swizzle)\w*|(global|buffer|flat|scratch)_load_(?!lds)\w+|s_(buffer_)?load_\w+)")


def asm_statements(text):
    """The argument lists of the inline assembly statements of a source."""
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, at, quoted = 1, m.end(), False
        while depth:
            c = text[at]
            if c == "\\":
                at += 1
            elif c == '"':
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            at += 1
        yield text[m.end():at - 1]


def loads_without_a_wait(text):
    """Statements in which a load into registers is not followed by a wait: their outputs would count as written while the
    load is still under way, and the compiler may copy or spill them then."""
    out = []
    for statement in asm_statements(text):
        statement = re.sub(r"\\[nt]", " ", statement)
        last = None
        for m in LOAD.finditer(statement):
            last = m
        if last and "s_waitcnt" not in statement[last.end():]:
            out.append(statement)
    return out


@pytest.mark.parametrize("name", SOURCES)
def test_inline_assembly_waits_for_what_it_loads(name):
    with open(os.path.join(CSRC, name)) as f:
        assert loads_without_a_wait(f.read()) == []


def test_the_check_finds_a_load_that_is_not_waited_for():
    late = 'asm volatile("s_waitcnt vmcnt(2)\\n\\tds_read_b64 %0, %1" : "=v"(near) : "v"(at)); asm("s_waitcnt lgkmcnt(0)" : "+v"(near));'
    good = 'asm volatile("ds_read_b32 %0, %1\\n\\ts_waitcnt lgkmcnt(0)" : "=v"(t) : "v"(at)); asm("global_load_lds_dwordx4 %0, %1" : : "v"(a), "s"(b));'
    assert len(loads_without_a_wait(late)) == 1
    assert loads_without_a_wait(good) == []


def test_kernels_that_address_lds_from_zero_have_no_static_lds(tmp_path):
    """The walk's tables are addressed from byte 0 of LDS on, where dynamic LDS starts in a kernel without static LDS."""
    obj = os.path.join(os.path.dirname(CSRC), "_build", "pvq_walk.hip.o")
    if not os.path.exists(obj):
        build.build()
    llvm = "/opt/rocm/llvm/bin"
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.run([f"{llvm}/llvm-objcopy", f"--dump-section=.hip_fatbin={bundle}", obj, str(tmp_path / "copy.o")], check=True)
    subprocess.run([f"{llvm}/clang-offload-bundler", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={bundle}",
                    f"--output={code}", "--unbundle"], check=True)
    notes = subprocess.run([f"{llvm}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    kernels = re.findall(r"\.group_segment_fixed_size:\s*(\d+).*?\.name:\s*(\S*(?:decode|gemv)_walk_kernel\S*)", notes, re.S)
    assert len(kernels) > 50
    assert [name for size, name in kernels if size != "0"] == []


def walk_notes(tmp_path):
    """What the compiler notes about the kernels of pvq_walk.hip."""
    obj = os.path.join(os.path.dirname(CSRC), "_build", "pvq_walk.hip.o")
    if not os.path.exists(obj):
        build.build()
    llvm = "/opt/rocm/llvm/bin"
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.run([f"{llvm}/llvm-objcopy", f"--dump-section=.hip_fatbin={bundle}", obj, str(tmp_path / "copy.o")], check=True)
    subprocess.run([f"{llvm}/clang-offload-bundler", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={bundle}",
                    f"--output={code}", "--unbundle"], check=True)
    return subprocess.run([f"{llvm}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout


def test_products_on_the_walk_keep_their_waves(tmp_path):
    """Registers decide how many workgroups of a product a unit holds (64 for eight waves a SIMD, 80 for six): with integers of
    up to two words the kernels with tiles of 16 rows have eight waves, those of 5 to 8 vectors in groups of up to 16 seven
    or eight, in groups of 32 with one word six.  (28672 x 8192 times five vectors, D = 16, K = 58: 148 us, with seven waves
    in tiles of 16 rows 195; 3001 x 11008, D = 32, K = 4: 20.8 us, with five waves 27.8.)"""
    kernels = re.findall(r"\.name:\s*\S*gemv_walk_kernelI((?:Li\d+E)+)E.*?\.vgpr_count:\s*(\d+)", walk_notes(tmp_path), re.S)
    found = {tuple(int(v) for v in re.findall(r"Li(\d+)E", name)): int(registers) for name, registers in kernels}
    most = {}
    for (D, W, DX, DA, DB, R, NV) in found:
        if W <= 2 and R == 16:
            most[D, W, DX, DA, DB, R, NV] = 64
        elif W <= 2 and NV == 2 and (D <= 16 or W == 1):
            most[D, W, DX, DA, DB, R, NV] = 72 if D <= 16 else 80
    assert len(most) > 10
    assert {k: found[k] for k in most if found[k] > most[k]} == {}


def test_encoders_of_groups_of_eight_keep_their_values_in_registers(tmp_path):
    """Eight waves a SIMD leave a lane 64 registers; what does not fit there goes to scratch memory and back."""
    obj = os.path.join(os.path.dirname(CSRC), "_build", "pvq_encode8.hip.o")
    if not os.path.exists(obj):
        build.build()
    llvm = "/opt/rocm/llvm/bin"
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.run([f"{llvm}/llvm-objcopy", f"--dump-section=.hip_fatbin={bundle}", obj, str(tmp_path / "copy.o")], check=True)
    subprocess.run([f"{llvm}/clang-offload-bundler", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={bundle}",
                    f"--output={code}", "--unbundle"], check=True)
    notes = subprocess.run([f"{llvm}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    kernels = re.findall(r"\.name:\s*(\S*encode8_kernel\S*).*?\.vgpr_count:\s*(\d+).*?\.vgpr_spill_count:\s*(\d+)", notes, re.S)
    assert len(kernels) > 50
    assert [name for name, registers, spilled in kernels if int(registers) > 64 or int(spilled) > 0] == []
    # 80 for the six waves that three workgroups of 512 lanes make
    halves = re.findall(r"\.name:\s*(\S*encode8_halves_kernel\S*).*?\.vgpr_count:\s*(\d+).*?\.vgpr_spill_count:\s*(\d+)", notes, re.S)
    assert len(halves) > 30
    assert [name for name, registers, spilled in halves if int(registers) > 80 or int(spilled) > 0] == []
