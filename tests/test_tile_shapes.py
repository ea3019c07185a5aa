"""The automatic shape of the multi-sweep tile kernel exists for every lattice
that the kernel may be asked for.  Host code only; no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1101_0876_amd")


def test_every_size_has_a_shape(tmp_path):
    exe = str(tmp_path / "tile_shapes")
    subprocess.run(["hipcc", "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-I", os.path.join(PKG, "csrc"),
                    "-c", os.path.join(ROOT, "tests", "native", "tile_shapes.cpp"), "-o", exe + ".o"], check=True)
    subprocess.run(["hipcc", "-o", exe, exe + ".o", os.path.join(PKG, "libpotts.so"), f"-Wl,-rpath,{PKG}"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines()
    assert out == [f"sizes {7 * 4095}"], out[:5]
