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


def notes(path, kernel, tmp_path):
    """The template arguments of every instance of a kernel -> its registers, LDS bytes and scratch bytes."""
    out = {}
    for n, blob in enumerate(code_objects(path)):
        if kernel.encode() not in blob:
            continue
        file = tmp_path / f"{n}.co"
        file.write_bytes(blob)
        text = subprocess.run([READELF, "--notes", str(file)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for part in text.split(".agpr_count:")[1:]:
            name = re.search(rf"\.name:\s+\S*\d{kernel}I(f|6__half)(\S*?)EEv", part)
            if not name:
                continue
            form = tuple(int(v) if kind == "i" else v == "1" for kind, v in re.findall(r"L([ib])(\d+)E", name.group(2) + "E"))
            value = lambda key: int(re.search(rf"\.{key}:\s+(\d+)", part).group(1))
            out[("float32" if name.group(1) == "f" else "float16", *form)] = {
                "registers": value("vgpr_count"), "lds": value("group_segment_fixed_size"), "scratch": value("private_segment_fixed_size"),
                "spilled": value("vgpr_spill_count")}
    return out


@pytest.fixture(scope="module")
def lib_path():
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not found")
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg.lib_path()


@pytest.fixture(scope="module")
def kernels(lib_path, tmp_path_factory):
    """(type, DP, FULL, THREADS, FINE) -> ..."""
    found = notes(lib_path, "encode_filter_kernel", tmp_path_factory.mktemp("co"))
    assert len(found) > 40
    return found


def test_appends_of_odd_sub_vectors_fill_a_compute_unit(lib_path, tmp_path):
    """Eight wavefronts per SIMD take at most 64 registers each."""
    found = {form: k for form, k in notes(lib_path, "encode_few_any_kernel", tmp_path).items() if form[1:] == (8, 0)}
    assert len(found) == 2 and all(k["registers"] <= 64 and not k["spilled"] for k in found.values()), found


def test_no_instance_spills(kernels):
    """A spilled register's reload in the pair loop waits for the key requests ahead of it."""
    assert not {form: k for form, k in kernels.items() if k["scratch"] or k["spilled"]}


SHIM = r"""
#include "encode_grid.h"
using namespace lookat;
extern "C" void choose(int heads, int m, long pairs, int dp, int key32, int *out)
{
    const EfGrid g = ef_grid(heads, m, pairs, dp, key32);
    out[0] = g.splits, out[1] = g.threads, out[2] = g.fine;
}
extern "C" long cost(int heads, int m, long pairs, int dp, int key32, int threads, int fine, long s)
{
    const long on_a_cu = ((heads * s + 7) / 8 * m + 31) / 32;      // the grid deals heads x splits to eight dies of 32 compute units
    return EfForm(dp, key32, threads, fine).cost(on_a_cu, ((pairs + s - 1) / s + 3) / 4);
}
extern "C" long least(int heads, int m, long pairs, int dp, int key32)      // over every split count up to one pair per wavefront
{
    long best = 1L << 62;
    for (int f = ef_has_large(dp) ? 0 : 1; f < (ef_has_fine(dp, key32) ? 3 : 2); ++f)
        for (long s = 1; s <= 1024; ++s) {
            const int threads = f ? 256 : 512;
            const long c = cost(heads, m, pairs, dp, key32, threads, f == 2, s);
            best = c < best ? c : best;
            if (s * (threads / 64) >= pairs)
                break;
        }
    return best;
}
extern "C" int resident(int dp, int threads, int fine) { return ef_resident(dp, threads, fine); }
"""


@pytest.fixture(scope="module")
def grid(tmp_path_factory):
    import ctypes
    folder = tmp_path_factory.mktemp("grid")
    (folder / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_10155_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover", "-shared", "-fPIC", "-I", csrc,
                    str(folder / "shim.cpp"), "-o", str(folder / "shim.so")], check=True)
    lib = ctypes.CDLL(str(folder / "shim.so"))
    for name in ("cost", "least"):
        getattr(lib, name).restype = ctypes.c_long
    long, integer = ctypes.c_long, ctypes.c_int
    lib.choose.argtypes = [integer, integer, long, integer, integer, ctypes.POINTER(integer)]
    lib.cost.argtypes = [integer, integer, long, integer, integer, integer, integer, long]
    lib.least.argtypes = [integer, integer, long, integer, integer]

    def choose(heads, m, pairs, dp, key32):
        out = (ctypes.c_int * 3)()
        lib.choose(heads, m, pairs, dp, key32, out)
        return tuple(out)
    lib.chosen = choose
    return lib


def test_the_choice_knows_how_many_workgroups_a_compute_unit_holds(kernels, grid):
    """512 registers per SIMD lane, handed out in eights, and 160 KB of LDS."""
    for (dtype, dp, full, threads, fine), k in kernels.items():
        on_a_simd = 512 // (-(-k["registers"] // 8) * 8)
        fits = min(on_a_simd // (threads // 256), 160 * 1024 // k["lds"])
        assert fits == grid.resident(dp, threads, fine), (dtype, dp, full, threads, fine, k)


def test_the_choice_is_the_cheapest_split(grid):
    """The few split counts that are looked at against all of them; a launch in two terms does not queue behind itself."""
    worst = 1.0
    for dp in (4, 8, 16, 32, 64):
        for key32 in (0, 1):
            for heads, m in ((1, 1), (2, 1), (1, 7), (2, 5), (2, 8), (12, 2), (25, 1), (12, 4), (25, 5), (32, 2), (40, 4), (12, 16), (25, 16),
                             (32, 8), (40, 10), (32, 16), (40, 32), (129, 1), (1000, 3), (65535, 32)):
                for pairs in (1, 2, 5, 13, 32, 63, 100, 128, 511, 2000, 16384, (1 << 29) - 1):
                    splits, threads, fine = grid.chosen(heads, m, pairs, dp, key32)
                    assert 1 <= splits <= 1024 and threads in (256, 512) and (threads == 256 or not fine)
                    got = grid.cost(heads, m, pairs, dp, key32, threads, fine, splits)
                    worst = max(worst, got / grid.least(heads, m, pairs, dp, key32))
                    if fine and dp == 64 and -(-heads // 8) * m <= 32:
                        assert -(-heads * splits // 8) * m <= 32, (key32, heads, m, pairs, splits)
    assert worst <= 1.04
