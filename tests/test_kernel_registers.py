"""Registers of the built FP64 step kernels: the occupancy their measured times rest on (reads the
library's own kernel metadata; no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_14933_amd import hexsv

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Demangled kernel name -> {vgprs, scratch} of the code objects in the library."""
    objcopy, readelf = (os.path.join(LLVM, t) for t in ("llvm-objcopy", "llvm-readelf"))
    if not (os.path.exists(hexsv.LIB_PATH) and os.path.exists(objcopy) and shutil.which("c++filt")):
        pytest.skip("library or LLVM tools not there")
    d = tmp_path_factory.mktemp("co")
    fat = str(d / "fatbin")
    subprocess.run([objcopy, "--dump-section", f".hip_fatbin={fat}", hexsv.LIB_PATH, os.devnull],
                   check=True)
    blob = open(fat, "rb").read()
    starts = [m.start() for m in re.finditer(b"\x7fELF", blob)]
    found = {}
    for i, (a, b) in enumerate(zip(starts, starts[1:] + [len(blob)])):
        co = d / f"co{i}"
        co.write_bytes(blob[a:b])
        notes = subprocess.run([readelf, "--notes", str(co)], capture_output=True, text=True).stdout
        for k in notes.split("- .agpr_count")[1:]:
            def num(field):
                return int(re.search(rf"\.{field}:\s+(\d+)", k).group(1))
            found[re.search(r"\.name:\s+(\S+)", k).group(1)] = {
                "vgprs": num("vgpr_count"), "scratch": num("private_segment_fixed_size")}
    names = list(found)
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True,
                           check=True).stdout.splitlines()
    return {re.sub(r"^void hexsv::|\(.*", "", p): found[n] for n, p in zip(names, plain)}


@pytest.mark.parametrize("kernel", ["k_step", "k_ens_step"])
@pytest.mark.parametrize("tile,vgprs", [("64, 4, 256", 72), ("64, 8, 256", 96),
                                        ("64, 16, 256", 128), ("128, 8, 256", 128)])
def test_plain_fp64_steps_keep_their_waves(kernels, kernel, tile, vgprs):
    """512 registers of a SIMD lane: seven, five, four and four waves per SIMD."""
    k = kernels[f"{kernel}<double, {tile}, false, false>"]
    assert k["vgprs"] <= vgprs and k["scratch"] == 0, k


@pytest.mark.parametrize("tile,scratch", [("64, 16, 1024", 128), ("64, 32, 1024", 320),
                                          ("128, 16, 1024", 320)])
def test_persistent_fp64_ensemble_spills_little(kernels, tile, scratch):
    """1024 threads leave 128 registers; 200 to 436 bytes of scratch a lane cost up to 46 %."""
    assert kernels[f"k_ensemble<double, {tile}>"]["scratch"] <= scratch


@pytest.mark.parametrize("tile,scratch", [("64, 16, 1024", 24), ("64, 32, 1024", 108),
                                          ("128, 16, 1024", 108)])
def test_persistent_fp32_ensemble_spills_little(kernels, tile, scratch):
    """124 bytes a lane cost 5 %."""
    assert kernels[f"k_ensemble<float, {tile}>"]["scratch"] <= scratch


@pytest.mark.parametrize("kernel", ["k_resident", "k_ens_resident"])
def test_viscous_fp32_on_chip_tile_is_inlined(kernels, kernel):
    """As a function of its own the step took its arguments and arrays through scratch memory."""
    assert kernels[f"{kernel}<float, 2, 1, true, true>"]["scratch"] == 0
