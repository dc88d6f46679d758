"""Vector registers of the kernels in the built library, from the metadata of its own code objects: how many wavefronts a SIMD
holds is decided by the largest of a kernel's bodies, so a body for the rare tiles can cost the others theirs."""

import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2410_11998_amd import build as bld

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects in the library's bundles, one for each translation unit with kernels."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if triple.endswith("gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def kernels(tmp_path):
    """{demangled name: (vector registers, bytes of scratch)}"""
    got = {}
    for k, obj in enumerate(code_objects(bld.LIB)):
        f = tmp_path / f"{k}.co"
        f.write_bytes(obj)
        text = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for entry in text.split("- .agpr_count:")[1:]:
            field = lambda name: re.search(r"\." + name + r":\s+(\S+)", entry).group(1)
            got[field("name")] = (int(field("vgpr_count")), int(field("private_segment_fixed_size")))
    names = list(got)
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True).stdout.splitlines()
    return {re.sub(r"dadam::|\(anonymous namespace\)::|void ", "", p).rsplit("(", 1)[0]: got[n] for n, p in zip(names, plain)}


def ceiling(name):
    """Registers up to which the kernel keeps the wavefronts per SIMD that it was measured with, None where that is not held."""
    m = re.match(r"(k_tile_few|k_tile|k_direct_few|k_direct)<(.*)>", name)
    if not m:
        return None
    a = m.group(2).split(", ")
    kind, xt, gt, phase = m.group(1), a[0], a[1], int(a[2])
    if not kind.endswith("few") and a[-1] == "true":        # tables in device memory: more registers for look-ups
        return None
    fold, plain, mixing = phase == 4, phase == 2, phase in (0, 6)
    if kind.startswith("k_tile"):
        vectors = int(a[4])
        if vectors == 2 and not mixing and (xt == "TBF16" or kind == "k_tile_few" or a[5] == "false"):
            return None                                     # steps take two vectors only where float32 streams
        if vectors == 2 and xt == "TBF16":
            return 72
        if fold:
            return 64 if xt == "TF32" and vectors == 1 else 72
        return 72 if xt == "TBF16" and gt == "TF32" and plain else 64
    if xt == "TBF16":
        return 64 if mixing else 96 if fold or plain else 80
    return 72 if fold or plain else 64


def test_registers_and_scratch_of_the_kernels(tmp_path):
    if not os.path.exists(f"{LLVM}/llvm-readelf") or shutil.which("c++filt") is None:
        pytest.skip("no llvm-readelf or c++filt")
    found = kernels(tmp_path)
    assert len(found) > 900 and "k_tile<TF32, TF32, 2, 16, 2, true, false>" in found and "k_direct_few<TBF16, TF32, 3>" in found
    assert not [n for n, (_, scratch) in found.items() if scratch]
    held = {n: ceiling(n) for n in found if ceiling(n) is not None}
    assert len(held) > 250
    over = {n: (found[n][0], most) for n, most in held.items() if found[n][0] > most}
    assert not over, over


def test_kernels_of_layouts_with_a_map_hold_as_many_wavefronts(tmp_path):
    """Each stands for an ordinary kernel, whose registers are held above or were measured: 512 a lane, given out by eight, for at most eight wavefronts."""
    if not os.path.exists(f"{LLVM}/llvm-readelf") or shutil.which("c++filt") is None:
        pytest.skip("no llvm-readelf or c++filt")
    found = kernels(tmp_path)
    waves = lambda name: min(8, 512 // (-(-found[name][0] // 8) * 8))
    mapped = [n for n in found if "_map<" in n]
    assert len(mapped) > 900 and {n.split("<")[0] for n in mapped} == {
        "k_tile_map", "k_tile_few_map", "k_direct_map", "k_direct_few_map", "k_loop_map", "k_mix_rows_map", "k_acc_map", "k_acc_few_map"}
    fewer = {n for n in mapped if waves(n) < waves(n.replace("_map<", "<"))}
    # mixing with the error of more than 64 bfloat16 rows over at most 16 sources: seven
    assert fewer <= {f"k_tile_map<TBF16, {g}, 6, 4, 2, true, true>" for g in ("TF32", "TBF16")}, fewer
