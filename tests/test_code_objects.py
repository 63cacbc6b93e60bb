"""What the compiler made of the kernels, from the metadata of the library's code objects."""
import os
import re
import struct
import subprocess

import pytest

from paper_2506_04985_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The built library's code objects, one file per source."""
    if not os.path.exists(build.LIB):
        build.build()
    tmp = tmp_path_factory.mktemp("code_objects")
    fat = str(tmp / "fat")
    subprocess.check_call([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", build.LIB, str(tmp / "copy")])
    data, found = open(fat, "rb").read(), []
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):          # one per source file: entries of offset, size, length of name, name
        at, (entries,) = bundle.start() + 32, struct.unpack_from("<Q", data, bundle.start() + 24)
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            target, at = data[at + 24:at + 24 + length], at + 24 + length
            if b"gfx950" in target and size:
                found.append(str(tmp / f"co{len(found)}"))
                open(found[-1], "wb").write(data[bundle.start() + offset:bundle.start() + offset + size])
    assert found
    return found


@pytest.fixture(scope="module")
def kernels(code_objects):
    """name -> metadata text of every kernel of the built library."""
    found = {}
    for co in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", co], capture_output=True, text=True, check=True).stdout
        for text in notes.split("  - .agpr_count")[1:]:
            found[re.search(r"\.name:\s+(_Z\S+)\n", text).group(1)] = text
    return found


@pytest.fixture(scope="module")
def assembly(code_objects, kernels):
    """pattern -> {name: assembly} of the kernels whose names it matches."""
    def of(pattern):
        names, found = [n for n in kernels if re.search(pattern, n)], {}
        for co in code_objects:
            text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(names), co],
                                  capture_output=True, text=True, check=True).stdout
            for part in re.split(r"\n(?=[0-9a-f]+ <)", text)[1:]:
                found[re.match(r"[0-9a-f]+ <(\S+)>", part).group(1)] = part
        assert sorted(found) == sorted(names) and names
        return found
    return of


def test_arguments_of_the_static_quantizers_come_with_the_dispatch(kernels):
    """Fourteen words are preloaded; an argument beyond them that a wave needs early is a memory latency of its own."""
    seen = 0
    for name, text in kernels.items():
        if re.search(r"quantize_act_(wave_)?kernelILi\dELi[1-9]", name):
            explicit = [(int(o), int(s)) for o, s, kind in re.findall(r"\.offset:\s+(\d+)\n\s+\.size:\s+(\d+)\n\s+\.value_kind:\s+(\w+)", text) if not kind.startswith("hidden")]
            assert len(explicit) == 9 and all(o + s <= 56 for o, s in explicit), (name, explicit)
            seen += 1
    assert seen > 30


def test_arguments_that_addresses_need_come_with_the_dispatch(kernels):
    """The quantizers that cut a row into pieces divide by the pieces of a row before their first load.  Only eps, which the sum comes before, may lie beyond."""
    seen = 0
    for name, text in kernels.items():
        if re.search(r"quantize_act_(flat|hadamard|hadamard_group)_kernel", name):
            ends = [int(o) + int(s) for o, s, kind in re.findall(r"\.offset:\s+(\d+)\n\s+\.size:\s+(\d+)\n\s+\.value_kind:\s+(\w+)", text) if not kind.startswith("hidden")]
            late = 1 if "hadamard_kernel" in name else 0
            assert len(ends) == (9 if "group" in name else 10) and sum(e > 56 for e in ends) == late and ends[-1] <= 60, (name, ends)
            seen += 1
    assert seen == 18 + 40 + 4


def test_scratch_only_where_it_is_stated(kernels):
    """Of the instances that calls run: the six-bit 256-token tile of whole 16-byte rows."""
    stated = (r"linear_prefill_kernelILi8ELi[12]ELb0ELb[01]E",
              r"linear_(mfma|prefill)_kernel.*Li0ELb1ELb[01]E",                 # parity dumps of the accumulators
              r"linear_decode_kernelILi16ELi4ELi[24]E")                         # shapes that only fptq_set_decode_shape reaches
    for name, text in kernels.items():
        if int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", text).group(1)):
            assert any(re.search(s, name) for s in stated), name


def test_no_step_of_an_unrolled_loop_is_there_twice(assembly):
    """INT8 tiles with K groups: a launch turns the loop so seldom that the time in which code arrives counts, so the steps left over are not copies of their own."""
    for name, text in assembly(r"linear_mfma_kernelINS_7GemmCfgI(Li\dE){5}Li1ELi[24]ELb[01]EEELi[012]ELb0E").items():
        wn, wm, tn, tm, stages = (int(v) for v in re.search(r"GemmCfgILi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)E", name).groups())
        assert text.count("v_mfma") == stages * 4 * tn * tm, name


def test_accumulators_are_set_once(assembly):
    for name, text in assembly(r"linear_mfma_kernelINS_7GemmCfg\w*EEELi2ELb0ELb0E").items():
        tn, tm = (int(v) for v in re.search(r"GemmCfgILi\dELi\dELi(\d)ELi(\d)E", name).groups())
        before = text[:text.index("v_mfma")]
        assert len(re.findall(r"v_accvgpr_write_b32 a\d+, 0\b|v_mov_b32_e32 v\d+, 0\b", before)) < 1.5 * 16 * tn * tm, name


def test_few_k_tiles_run_little_code(assembly):
    """The six-bit kernel of up to 32 K tiles: two steps' code, and one for what is left over."""
    found = assembly(r"linear_prefill_kernelILi[68]E\w*ELi2EEEv")
    assert len(found) == 16
    for name, text in found.items():
        assert text.count("v_mfma") == 3 * 4 * int(re.search(r"ILi(\d)E", name).group(1)), name
