"""Compiles small programs against the host-only headers of csrc/ with the system compiler."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_12780_amd", "csrc")


def compile_cpp(directory, source):
    src, exe = os.path.join(directory, "t.cpp"), os.path.join(directory, "t")
    with open(src, "w") as f:
        f.write(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", CSRC, src, "-o", exe], check=True)
    return exe


def run(exe, text=""):
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
