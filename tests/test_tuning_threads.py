"""The launch-shape table under several threads: storing one form's part count never
undoes another thread's update of the entry."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_counts_of_the_two_forms_are_stored_independently(tmp_path):
    exe, lib = os.path.join(tmp_path, "tuning_threads"), os.path.join(ROOT, "paper_1807_10151_amd")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "c_abi", "tuning_threads.cpp"), "-L", lib, "-lsuppcg",
                    f"-Wl,-rpath,{lib}", "-Wl,--allow-shlib-undefined"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and int(res.stdout) == 0, res.stdout + res.stderr
