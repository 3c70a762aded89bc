"""Tickets, rings and prefixes of the encode kernel as a simulation over the kernel's own rules: no count is stored over a prefix
and all waits end, in every tile order, with few workers and with workers that start late."""
import os
import subprocess
import tempfile

from test_host_sanitizers import ROOT, SAN, run


def test_walk_under_every_order():
    csrc = os.path.join(ROOT, "paper_2605_06534_amd", "csrc")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "walk_driver")
        subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Wextra"] + SAN +
                              ["-I", os.path.join(ROOT, "include"), "-I", csrc,
                               os.path.join(ROOT, "tests", "sanitize", "walk_driver.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe])
        run(exe)
