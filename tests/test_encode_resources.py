"""What the compiler gave the ranking encoder's kernels, read from the built library's kernel descriptions."""
import os
import re
import shutil
import struct
import subprocess

import pytest

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects in a library, one per translation unit."""
    data = open(path, "rb").read()
    for found in re.finditer(MAGIC, data):
        at = found.start() + len(MAGIC)
        count, at = struct.unpack_from("<Q", data, at)[0], at + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name:
                yield data[found.start() + offset:found.start() + offset + size]


def encoder_kernels(path, tmp_path):
    """(type, DP, FULL, THREADS, FINE) -> registers, LDS bytes and scratch bytes of every encode_filter_kernel instance."""
    out = {}
    for n, blob in enumerate(code_objects(path)):
        if b"encode_filter_kernel" not in blob:
            continue
        file = tmp_path / f"{n}.co"
        file.write_bytes(blob)
        text = subprocess.run([READELF, "--notes", str(file)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for part in text.split(".agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S*encode_filter_kernel\S*)", part)
            if not name:
                continue
            form = re.search(r"kernelI(f|6__half)Li(\d+)ELb(\d)ELi(\d+)ELb(\d)E", name.group(1)).groups()
            value = lambda key: int(re.search(rf"\.{key}:\s+(\d+)", part).group(1))
            out[("float32" if form[0] == "f" else "float16", int(form[1]), form[2] == "1", int(form[3]), form[4] == "1")] = {
                "registers": value("vgpr_count"), "lds": value("group_segment_fixed_size"), "scratch": value("private_segment_fixed_size"),
                "spilled": value("vgpr_spill_count")}
    return out


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not found")
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    found = encoder_kernels(pkg.lib_path(), tmp_path_factory.mktemp("co"))
    assert len(found) > 40
    return found


def test_no_instance_spills(kernels):
    """A spilled register's reload in the pair loop waits for the key requests ahead of it."""
    assert not {form: k for form, k in kernels.items() if k["scratch"] or k["spilled"]}
