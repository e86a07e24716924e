"""What the compiler made of the sweep kernels, read from the built library:
no kernel keeps registers in memory, and none holds copies of registers where
lanes that should make them are off."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

import paper_2002_00352_amd as kp

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def _code_objects(tmp):
    """The gfx950 code objects of libkp.so (the offload bundles of its fat binary section)."""
    fat = os.path.join(tmp, "fat")
    subprocess.check_call([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", f".hip_fatbin={fat}", kp.LIB_PATH,
                           os.path.join(tmp, "copy")])
    data = open(fat, "rb").read()
    out, pos = [], data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while pos >= 0:
        n, at = struct.unpack_from("<Q", data, pos + 24)[0], pos + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if "gfx950" in name and size:
                out.append(os.path.join(tmp, f"object{len(out)}"))
                open(out[-1], "wb").write(data[pos + off:pos + off + size])
        pos = data.find(b"__CLANG_OFFLOAD_BUNDLE__", pos + 24)
    return out


def _kernels(path):
    """The kernels' metadata (the AMDGPU note of a code object)."""
    elf = open(path, "rb").read()
    phoff, = struct.unpack_from("<Q", elf, 32)
    size, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        kind, _, off, _, _, length = struct.unpack_from("<IIQQQQ", elf, phoff + i * size)
        if kind != 4:   # PT_NOTE
            continue
        at = off
        while at < off + length:
            nsz, dsz, ntype = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (nsz + 3) // 4 * 4
            if ntype == 32:
                return msgpack.unpackb(elf[desc:desc + dsz])["amdhsa.kernels"]
            at = desc + (dsz + 3) // 4 * 4
    return []


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    if not (os.path.exists(kp.LIB_PATH) and os.path.exists(os.path.join(LLVM, "llvm-objdump"))):
        pytest.skip("needs the built library and the ROCm LLVM tools")
    objs = _code_objects(str(tmp_path_factory.mktemp("objects")))
    assert objs
    return objs


def test_sweep_kernels_need_no_scratch(objects):
    found, spilling = 0, []
    for path in objects:
        for k in _kernels(path):
            if re.search(r"k_(ell|dense|sweep|sel|scd|fix)", k[".name"]):
                found += 1
                if k[".private_segment_fixed_size"]:
                    spilling.append((k[".name"], k[".private_segment_fixed_size"]))
    assert found > 100
    assert not spilling, spilling


def test_no_register_copies_under_a_stale_lane_mask(objects):
    """A copy to a spill register at the head of a block that then restores the
    lane mask runs only in the lanes of the branch before it: after a branch
    that no lane took it does nothing, and the register is stale."""
    bad, blocks = [], 0
    for path in objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--symbolize-operands", path],
                              check=True, capture_output=True, text=True).stdout
        kernel, copies = None, None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                kernel = kernel if re.fullmatch(r"L\d+", m.group(1)) else m.group(1)
                copies, blocks = 0, blocks + 1
                continue
            op = line.strip()
            if copies is None or not op:
                continue
            if re.match(r"s_or_b64 exec, exec|s_or_saveexec|s_mov_b64 exec", op):
                if copies:
                    bad.append((kernel, copies))
                copies = None
            elif re.match(r"v_accvgpr_write|v_accvgpr_mov|scratch_store|buffer_store.*offen", op):
                copies += 1
            elif op.startswith(("s_cbranch", "s_branch", "s_endpgm")) or "exec" in op.split("//")[0]:
                copies = None
    assert blocks > 1000
    assert not bad, bad
