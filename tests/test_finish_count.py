"""The count by which a one-launch reduction finds its last workgroup, on the CPU: it also holds after launches that overlapped."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_last_workgroup_is_found_also_after_overlapping_launches(tmp_path):
    exe = str(tmp_path / "finish_count")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1811_09736_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "sanitize", "finish_count_driver.cpp")], check=True)
    assert subprocess.run([exe], stdout=subprocess.PIPE, text=True, check=True).stdout.strip().endswith("ok")
