"""The sliced rows of large levels on the CPU: the stored layout against a
brute-force look at the rows, tiles cut for their dictionaries, and the rule
that keeps uneven or scattered rows in dictionary tiles
(tests/cpp/sliced_layout_check.cpp with csrc/setup.cpp, the library's flags)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_sliced_rows_of_even_uneven_and_scattered_matrices(tmp_path):
    exe = str(tmp_path / "sliced_layout_check")
    csrc = os.path.join(ROOT, "paper_2210_16660_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-ffp-contract=off", "-fno-fast-math",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "cpp", "sliced_layout_check.cpp"),
                    os.path.join(csrc, "setup.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("0 failures")
