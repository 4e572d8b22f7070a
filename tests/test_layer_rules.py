"""Host-side rules of the layer kernels (CPU only): a small C++ program checks the library's arithmetic against plain loops."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2102_08481_amd")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")
def test_layer_kernels_host_arithmetic(tmp_path):
    """FastDiv and tap_mask against division and loops; every tap offset of the large tiles' buffer loads within 31 bits for all
    layer forms that they accept, near the limit in particular."""
    if not os.path.exists(os.path.join(PKG, "libthia.so")):
        from paper_2102_08481_amd import build
        build.build()
    exe = str(tmp_path / "layer_rules_driver")
    r = subprocess.run(["hipcc", "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-O2", "-std=c++17",
                        os.path.join(PKG, "csrc", "layer_rules_driver.cpp"), "-o", exe, "-L" + PKG, "-lthia", "-Wl,-rpath," + PKG],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "layer_rules_driver: ok" in r.stdout, r.stdout[-4000:] + r.stderr[-2000:]
