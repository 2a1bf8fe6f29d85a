"""Registers and scratch of the compiled kernels, read from the metadata of the objects that the build leaves: what a
change of the source costs here shows in no result.  CPU only."""
import os
import re
import subprocess

import pytest

from paper_2512_18453_amd import build

TOOLS = "/opt/rocm/llvm/bin"


def resources(source, tmp_path):
    obj = os.path.join(build.OBJ, source + ".o")
    if not os.path.exists(obj):
        pytest.skip("objects are not built here")
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.check_call(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", "--set-section-flags", ".hip_fatbin=alloc", obj, bundle])
    subprocess.check_call([f"{TOOLS}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                           f"--input={bundle}", f"--output={code}"])
    notes = subprocess.check_output([f"{TOOLS}/llvm-readelf", "--notes", code], text=True)
    names = [ln.split()[1] for ln in notes.splitlines() if ln.startswith("    .name:")]
    plain = subprocess.run(["c++filt"], input="\n".join(n.replace("DF16_", "Dh") for n in names), capture_output=True, text=True, check=True)

    def every(field):
        return [int(v) for v in re.findall(rf"^    \.{field}: +(\d+)$", notes, re.M)]
    keys = [re.search(r"(\w+<.*?>)\(", p)[1].replace("false", "0").replace("true", "1") for p in plain.stdout.splitlines()]
    return dict(zip(keys, zip(every("vgpr_count"), every("private_segment_fixed_size"), strict=True), strict=True))


def test_input_transform(tmp_path):
    # <n, r, type, paired points, channels, wide, streaming, maxima>; three waves per SIMD have 168 registers each
    got = resources("input_transform.hip", tmp_path)
    for r in (3, 5):
        for stream in (0, 1):
            registers, scratch = got[f"input_transform_kernel<10, {r}, half, 1, 32, 0, {stream}, 0>"]
            assert registers <= 136 and scratch == 0, (r, stream, registers, scratch)
        assert got[f"input_transform_kernel<10, {r}, half, 1, 4, 0, 0, 0>"][0] <= 136
    assert all(scratch == 0 for name, (_, scratch) in got.items() if not re.search("<10, ., half, 1, 32, 0, 0, [12]>", name))


def test_one_kernel_layers(tmp_path):
    # <n, r, type, tiles, output channels, threads per tile and word, ReLU, rows first>: the variants known to spill, and no more
    spills = {("8", "half", "16"): 44, ("10", "half", "8"): 20, ("10", "float", "8"): 108}
    for name, (_, scratch) in resources("layer.hip", tmp_path).items():
        n, _, dtype, tiles = re.findall(r"[\w.]+", name)[1:5]
        assert scratch <= spills.get((n, dtype, tiles), 0), name


def test_contraction_and_output_in_one_kernel(tmp_path):
    # <n, r, 64-channel stages, ring, workgroups per unit, streaming>
    scratch = {("8", "3", "1"): 32, ("8", "3", "2"): 28, ("10", "5", "1"): 48, ("10", "5", "2"): 36, ("10", "5", "3"): 40}
    for name, (registers, spilled) in resources("contract_output.hip", tmp_path).items():
        n, r, chunks, _, per_unit = re.findall(r"[\w.]+", name)[1:6]
        assert spilled <= scratch.get((n, r, chunks), 0) and registers <= (256 if per_unit == "2" else 168), name
