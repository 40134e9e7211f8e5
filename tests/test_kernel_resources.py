"""Kernels keep their working set in registers: what a spill costs is memory traffic that no table of bytes accounts for."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2311_02909_amd", "libbms.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
KERNELS = ["feature_fetch_kernel", "dd_bitmap_kernel", "ldw_extract_kernel", "aggregate_kernel"]


def _code_objects(tmp_path):
    """the gfx950 code objects in the library, as files"""
    data = open(LIB, "rb").read()
    objects = []
    at = data.find(MAGIC)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(entries):
            offset, size, name_len = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + name_len].decode()
            p += 24 + name_len
            if "gfx950" not in name or not size:
                continue
            objects.append(tmp_path / ("code%d" % len(objects)))
            objects[-1].write_bytes(data[at + offset:at + offset + size])
        at = data.find(MAGIC, at + 1)
    return objects


def _readelf(what, obj):
    return subprocess.run([READELF, what, "--wide", str(obj)], check=True, capture_output=True, text=True).stdout


def _scratch_bytes(tmp_path):
    """kernel name -> bytes of scratch per lane, from the notes of the code objects"""
    found = {}
    for obj in _code_objects(tmp_path):
        for kernel in re.split(r"\n\s*- \.", _readelf("--notes", obj)):
            name = re.search(r"\.?name:\s+(_ZN3bms\S+)\n", kernel)
            bytes_ = re.search(r"private_segment_fixed_size:\s+(\d+)", kernel)
            if name and bytes_:
                found[name.group(1)] = int(bytes_.group(1))
    return found


def _code_bytes(tmp_path):
    """kernel name -> bytes of its instructions"""
    return {name: int(size) for obj in _code_objects(tmp_path)
            for size, name in re.findall(r"\s(\d+)\s+FUNC\s.*\s(_ZN3bms\S+)\n", _readelf("--dyn-syms", obj))}


@pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(READELF)), reason="library or tools not here")
@pytest.mark.parametrize("kernel", KERNELS)
def test_kernel_does_not_spill(kernel, tmp_path):
    found = {name: size for name, size in _scratch_bytes(tmp_path).items() if kernel in name}
    assert found and not any(found.values())


# a launch that does not go by dies, as those of small hops, carries nothing of that walk, which is two kilobytes of instructions
@pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(READELF)), reason="library or tools not here")
def test_sampling_in_stacked_order_has_kernels_of_its_own(tmp_path):
    size = {name: n for name, n in _code_bytes(tmp_path).items() if "nw_sample_kernelILi" in name}
    stacked = [name for name in size if "ELb0EEEv" in name]
    assert len(stacked) == 40 and len(size) == 80
    for name in stacked:
        assert size[name] + 1000 < size[name.replace("ELb0EEEv", "ELb1EEEv")], name


# the workgroup that is done last sets its counter back, waits until that is where the next call's kernels find it, and only then tells
# the host, which may make that call on another stream at once
@pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(OBJDUMP)), reason="library or tools not here")
def test_a_call_is_announced_behind_the_counter_of_its_workgroups(tmp_path):
    kernel = "_ZN3bms24ldw_extract_place_kernelILb1EEEvNS_5LwHopENS_8LookbackEPlNS_11PublishArgsE"
    for obj in _code_objects(tmp_path):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + kernel, str(obj)], check=True,
                              capture_output=True, text=True).stdout
        if kernel + ">:" not in text:
            continue
        code = [line.split("//")[0].strip() for line in text.splitlines()]
        added, = [x for x, line in enumerate(code) if line.startswith("global_atomic_add ") and " sc0" in line and
                  any(other.startswith("s_endpgm") for other in code[x:x + 40])]
        tail = [line for line in code[added:] if line.startswith(("global_store", "s_waitcnt vmcnt(0)"))]
        assert [line.split()[0] for line in tail] == ["s_waitcnt", "global_store_dword", "s_waitcnt", "global_store_dwordx2"], tail
        return
    raise AssertionError("kernel not found")
