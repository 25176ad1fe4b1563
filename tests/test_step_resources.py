"""What the compiler gave the fused steps' kernels, read from the built library's kernel descriptions."""
import re
import subprocess

from test_encode_resources import READELF, code_objects, lib_path  # noqa: F401


def instances(path, tmp_path):
    """(head size, subspaces, type, query heads) of the fused instances of decode_split_kernel -> registers, spilled registers."""
    out = {}
    for n, blob in enumerate(code_objects(path)):
        if b"decode_split_kernel" not in blob:
            continue
        file = tmp_path / f"{n}.co"
        file.write_bytes(blob)
        text = subprocess.run([READELF, "--notes", str(file)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for part in text.split(".agpr_count:")[1:]:
            name = re.search(r"\.name:\s+\S*decode_split_kernelILi(\d+)ELi(\d+)ELi\d+ELi\d+E(f|6__half)Li(\d+)E", part)
            if name:
                value = lambda key: int(re.search(rf"\.{key}:\s+(\d+)", part).group(1))
                form = (int(name.group(1)), int(name.group(2)), "float32" if name.group(3) == "f" else "float16", int(name.group(4)))
                out.setdefault(form, []).append((value("vgpr_count"), value("vgpr_spill_count")))
    return out


def test_two_workgroups_of_four_heads_share_a_compute_unit(lib_path, tmp_path):  # noqa: F811
    """Eight wavefronts each, four to a SIMD: 128 registers.  With 132 launches of more than 256 workgroups took up to 1.13 times as long."""
    found = {form: regs for form, regs in instances(lib_path, tmp_path).items() if form[0] == 64 and form[3] == 4}
    assert len(found) == 8
    assert all(registers <= 128 and not spilled for regs in found.values() for registers, spilled in regs), found
