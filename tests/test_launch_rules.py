"""Rules by which the library lays out and admits launches, checked on the CPU:
their headers hold no device code and compile with the host compiler."""

import os
import shutil
import subprocess

import pytest

RULES = os.path.join(os.path.dirname(os.path.abspath(__file__)), "rules")


def _run_driver(tmp_path_factory, name):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("rules") / name)
    p = subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", os.path.join(RULES, name + ".cpp"),
                        "-o", out], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    p = subprocess.run([out], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                       timeout=120)
    assert p.returncode == 0, p.stdout
    return p.stdout


def test_persistent_runs_admitted_together_are_resident(tmp_path_factory):
    # Blocks of persistent solves wait for each other: mixed block sizes, block
    # counts that do not divide among the XCDs, any placement, runs in order.
    _run_driver(tmp_path_factory, "residency_driver")


def test_launch_rules(tmp_path_factory):
    _run_driver(tmp_path_factory, "rules_driver")
