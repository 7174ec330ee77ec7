"""The search kernels of the paper's row width keep everything in registers: a kernel that spills uses scratch
memory, and a launch of one takes about 2 us longer to start.  Read from the kernel descriptions in the built library."""
import os
import re
import struct
import subprocess

import pytest

import paper_2503_10017_amd as fnn

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def scratch_bytes(tmp_path):
    """Kernel name -> bytes of scratch memory per lane, over every gfx950 code object in the library."""
    return {name: scratch for name, (scratch, _) in kernel_notes(tmp_path).items()}


def code_objects(tmp_path):
    """Every gfx950 code object in the library, each as a file."""
    with open(fnn.library_path(), "rb") as f:
        image = f.read()
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", image):
        at = bundle.end()
        count, = struct.unpack_from("<Q", image, at)
        at += 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", image, at)
            target = image[at + 24:at + 24 + name_len]
            at += 24 + name_len
            if b"gfx950" not in target or size == 0:
                continue
            path = tmp_path / "code.o"
            path.write_bytes(image[bundle.start() + offset:bundle.start() + offset + size])
            yield str(path)


def kernel_notes(tmp_path):
    """Kernel name -> (bytes of scratch memory per lane, vector registers)."""
    found = {}
    for path in code_objects(tmp_path):
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
        for name, scratch, rest in re.findall(r"\.name:\s+(_Z\S+)\n\s+\.private_segment_fixed_size: (\d+)\n((?:\s+\.(?!name:|args:).*\n)*)", notes):
            found[name] = int(scratch), int(re.search(r"\.vgpr_count:\s+(\d+)", rest).group(1))
    return found


@pytest.mark.parametrize("kernel", ["search_kernel", "search_first_kernel"])
def test_no_scratch_memory_at_24_channels_in_16_bits(kernel, tmp_path):
    scratch = scratch_bytes(tmp_path)
    half24 = {k: v for k, v in scratch.items()
              if re.match(rf"_ZN3fnn\d+{kernel}ILi[12]E" + ("Li24E" if kernel == "search_kernel" else ""), k)}
    assert len(half24) >= 2
    assert not {k: v for k, v in half24.items() if v}


def test_no_scratch_memory_in_the_8_bit_passes(tmp_path):
    scratch = scratch_bytes(tmp_path)
    for kernel, count in (("coarse_kernel", 5), ("dense_coarse_kernel", 2), ("dense_select_kernel", 1), ("dense_sample_kernel", 1), ("dense_judge_kernel", 1)):
        found = {k: v for k, v in scratch.items() if re.match(rf"_ZN3fnn\d+{kernel}[IE]", k)}
        assert len(found) == count, (kernel, sorted(found))
        assert not {k: v for k, v in found.items() if v}
    for kernel in ("refine_kernel", "quantise_kernel"):   # 16-bit rows of 24 channels
        found = {k: v for k, v in scratch.items() if re.match(rf"_ZN3fnn\d+{kernel}ILi[12]ELi24E", k)}
        assert len(found) >= 4 and not {k: v for k, v in found.items() if v}


def test_scratch_memory_of_the_late_iterations(tmp_path):
    """None for rows of up to 96 bytes; wider ones keep a few registers there, which costs less than fewer query blocks would."""
    found = {k: v for k, v in scratch_bytes(tmp_path).items() if re.match(r"_ZN3fnn\d+recip_tail_kernelI", k)}
    assert len(found) == 14
    for name, scratch in found.items():
        compute, channels = (int(x) for x in re.match(r".*recip_tail_kernelILi(\d)ELi(\d+)E", name).groups())
        row_bytes = channels * (4 if compute == 0 else 2)
        assert scratch <= (0 if row_bytes <= 96 else (32 if row_bytes <= 160 else 96)), (name, scratch)


def test_workgroups_that_the_choice_between_whole_and_half_segments_counts_on(tmp_path):
    """A workspace is sized without a device, so the rule has the resident workgroups of coarse_kernel's variants as numbers: four waves each, one
    on every SIMD of 256 compute units (the stages' 16 KB of LDS leave room for ten)."""
    with open(os.path.join(os.path.dirname(fnn.__file__), "csrc", "coarse.hip")) as f:
        source = f.read()
    said = {8: "COARSE_WGS_8", 6: "COARSE_WGS_6", 2: "COARSE_WGS_HALF"}
    said = {pairs: int(re.search(rf"{name} = (\d+)[,;]", source).group(1)) for pairs, name in said.items()}
    seen = set()
    for name, (_, registers) in kernel_notes(tmp_path).items():
        of = re.match(r"_ZN3fnn\d+coarse_kernelILi(\d)E", name)
        if of:
            seen.add(int(of.group(1)))
            assert 256 * (512 // (-(-registers // 8) * 8)) == said[int(of.group(1))], (name, registers)
    assert seen == set(said)


def test_what_workgroups_hand_each_other_passes_the_caches_of_their_xcds(tmp_path):
    """The late iterations' shared words are read and written by instructions with the sc1 bit; what has none is a fragment of a map (16 bytes, or 16 and 8) or one
    of the three results, in the two places that write them."""
    kernels = 0
    for path in code_objects(tmp_path):
        with open(path, "rb") as f:
            if b"recip_tail_kernel" not in f.read():
                continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout
        for name, body in re.findall(r"<(_ZN3fnn\d+recip_tail_kernel\w+)>:\n(.*?)(?=\n\n|\Z)", text, re.S):
            kernels += 1
            plain = [op for op, rest in re.findall(r"^\s+((?:global|flat|buffer)_(?:load|store)\w*)\s+(.*)$", body, re.M) if "sc1" not in rest]
            assert {op for op in plain if "load" in op} <= {"global_load_dwordx4", "global_load_dwordx2"}, name
            eight = plain.count("global_load_dwordx2")
            assert eight == (plain.count("global_load_dwordx4") if re.search(r"ILi[12]ELi24E", name) else 0), name
            assert [op for op in plain if "store" in op] == ["global_store_dword"] * 6, name
    assert kernels == 14
