"""What the compiler made of the kernels, read from the code objects inside the built library: properties that cost
time and not correctness when they are lost, and that no result shows."""
from __future__ import annotations

import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2510_11400_amd", "libfedhybrid.so")
LLVM = "/opt/rocm/lib/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """Paths of the device code objects of the library: one bundle per source file."""
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    out = tmp_path_factory.mktemp("code")
    with open(LIB, "rb") as f:
        data = f.read()
    magic, paths = b"__CLANG_OFFLOAD_BUNDLE__", []
    for m in re.finditer(magic, data):
        at = m.start() + len(magic)
        (entries,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name and size:
                paths.append(str(out / f"{len(paths)}.o"))
                with open(paths[-1], "wb") as f:
                    f.write(data[m.start() + offset:m.start() + offset + size])
    assert len(paths) >= 6, "the library's code objects were not found"
    return paths


def _disassembly(paths, function):
    """{demangled name: [instructions]} of the functions whose name contains `function`."""
    found = {}
    for p in paths:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--demangle", "--no-show-raw-insn", p], check=True,
                              capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            head = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if head:
                name = head.group(1) if function in head.group(1) else None
            elif name and line.strip():
                found.setdefault(name, []).append(line.split("//")[0].strip())
    return found


def _resources(paths):
    """{mangled name: its entry in the code objects' notes}"""
    found = {}
    for p in paths:
        text = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", p], check=True, capture_output=True, text=True).stdout
        for entry in text.split("  - .agpr_count:")[1:]:
            values = dict(re.findall(r"^    \.(\w+):\s+(\S+)$", entry, re.M))
            found[values["symbol"].strip("'").removesuffix(".kd")] = {k: int(v) for k, v in values.items() if v.isdigit()}
    return found


def test_no_kernel_needs_scratch_memory(code_objects):
    """A register bound that the compiler meets by spilling costs more than the waves or the loads in flight it buys."""
    kernels = _resources(code_objects)
    assert len(kernels) >= 80
    for name, r in kernels.items():
        assert r["vgpr_spill_count"] == 0 and r["private_segment_fixed_size"] == 0, f"{name}: {r}"


def test_launches_of_one_tensor_have_short_arguments(code_objects):
    """Up to 112 bytes of arguments a launch is enqueued a microsecond sooner; a hidden argument (the grid's size, for
    one) would make the segment some 300 bytes long."""
    kernels = {name: r for name, r in _resources(code_objects).items() if "_one_kernel" in name or "3OneI" in name}
    families = {re.search(r"\d([a-z_]+_kernel)", name).group(1) for name in kernels}
    assert families == {"compress_one_kernel", "decompress_one_kernel", "compress_mixed_one_kernel", "decompress_mixed_one_kernel",
                        "moments_one_kernel", "reduce_partials_kernel", "count_outliers_kernel", "count_marked_kernel", "mask_kernel",
                        "compress_first_kernel", "chain_prepare_kernel", "huffman_histogram_kernel", "huffman_code_kernel",
                        "huffman_count_kernel", "huffman_write_kernel", "huffman_decode_kernel"}
    for name, r in kernels.items():
        assert r["kernarg_segment_size"] <= 112, f"{name}: {r['kernarg_segment_size']}"


def test_the_rows_of_a_wave_are_requested_together(code_objects):
    """The classification's first pass: a wave's whole rows are read by non-temporal 16-byte loads with no wait for
    one of them before the last is on its way (a test around each row's load makes the compiler wait for the first, which
    only the form for large launches of fp32 is better off with)."""
    kernels = _disassembly(code_objects, "moments_kernel<")
    assert len(kernels) == 4
    kernels = {name: code for name, code in kernels.items() if "moments_kernel<float, true>" not in name}
    assert len(kernels) == 3
    for name, code in kernels.items():
        rows = [i for i, op in enumerate(code) if op.startswith("global_load_dwordx4") and op.endswith(" nt")]
        assert len(rows) in (2, 4), f"{name}: {len(rows)} row loads"
        waits = [op for op in code[rows[0]:rows[-1]] if op.startswith("s_waitcnt") and "vmcnt" in op]
        assert not waits, f"{name}: {waits} between the row loads"


def test_no_64_bit_shift_by_the_last_register(code_objects):
    """A 64-bit shift whose amount sits in the last vector register that a wave has been given was seen to shift by
    register 0 instead (the amount is read as a pair, and the pair leaves the allocation): the compiler does not avoid it."""
    kernels = _resources(code_objects)
    seen = 0
    for p in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", p], check=True,
                              capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            head = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if head:
                name = head.group(1)
                continue
            shift = re.search(r"v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\S*\s+v\[\d+:\d+\], v(\d+),", line)
            if shift and name in kernels:
                seen += 1
                given = -(-kernels[name]["vgpr_count"] // 8) * 8          # registers come in eights
                assert int(shift.group(1)) != given - 1, f"{name}: {line.split('//')[0].strip()}"
    assert seen > 0
