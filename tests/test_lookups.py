"""Index arithmetic that every attention address depends on: divisions as products (both sides of the bound up to which they
are exact, block sizes that are no powers of two, the largest rings), and the two-level search of an item's run."""
import os
import subprocess

import paper_2604_19769_amd

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.dirname(os.path.abspath(paper_2604_19769_amd.__file__))


def test_products_and_search_against_divisions_and_linear_search(tmp_path):
    exe = str(tmp_path / "lookups")
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I" + os.path.join(PKG, "..", "include"),
                    "-I" + os.path.join(PKG, "csrc"), os.path.join(HERE, "lookups.cpp"), "-L" + PKG, "-lttkv", "-Wl,-rpath," + PKG,
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
