"""The size limit of the sliced-ELL layout, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_limit_counts_entries_alone(tmp_path):
    exe = str(tmp_path / "check")
    host = os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", os.path.join(ROOT, "tests", "sell_offsets_check.cpp"),
                    os.path.join(host, "formats.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.returncode
