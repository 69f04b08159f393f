"""What the compiler gave the gated propagation kernels, read from the metadata of the built objects (no GPU): their throughput is the
number of wavefronts that are resident."""
import os
import re
import subprocess

import paper_1810_08403_amd.build as saga_build

LLVM = "/opt/rocm/llvm/bin"


def _kernels(obj, tmp):
    """{kernel: {attribute: value}} of the gfx950 code in an object of this library."""
    out = os.path.join(tmp, "code.co")
    sections = os.path.join(tmp, "fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={sections}", obj, os.path.join(tmp, "copy.o")], check=True)
    names = subprocess.run([f"{LLVM}/clang-offload-bundler", "--list", "--type=o", f"--input={sections}"], check=True, capture_output=True, text=True).stdout
    target = next(l for l in names.split() if "gfx950" in l)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--targets={target}", f"--input={sections}", f"--output={out}"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", out], check=True, capture_output=True, text=True).stdout
    kernels, now = {}, {}
    for line in notes.splitlines():
        m = re.match(r"\s+\.(name|vgpr_count|agpr_count|vgpr_spill_count|private_segment_fixed_size|symbol):\s+'?([\w.]+)'?", line)
        if not m:
            continue
        now[m.group(1)] = m.group(2)
        if m.group(1) == "vgpr_spill_count":          # (the last of a kernel's attributes)
            kernels[now["symbol"][:-3]] = {k: int(v) for k, v in now.items() if v.isdigit()}
            now = {}
    return kernels


def test_gated_propagation_keeps_its_wavefronts(tmp_path):
    obj = os.path.join(saga_build.OBJ_DIR, "gather.o")
    if not os.path.exists(obj):
        saga_build.build()
    kernels = _kernels(obj, str(tmp_path))
    # k_gather_narrow<float, 4, ragged, accumulator, gate>
    found = {n: k for n, k in kernels.items() if re.search(r"k_gather_narrowIfLi4ELb[01]ELi[01]ELi1EE", n)}
    assert len(found) == 4, sorted(kernels)[:20]
    for name, k in found.items():
        assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0, (name, k)
        assert k["vgpr_count"] <= (72 if "Lb1E" in name else 64), (name, k)    # seven and eight of 512 registers
