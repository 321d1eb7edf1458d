"""Runs a C++ program over the library's own headers on the CPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1603_06958_amd", "csrc")


def run(tmp_path, source, *args):
    src, exe = tmp_path / "prog.cpp", tmp_path / "prog"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, str(src), "-o", str(exe), "-lpthread"],
                   check=True)
    return subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True).stdout
