"""The context's workspace (dst_workspace.h) on the host, with a counting allocator."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("ws") / "workspace_check"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1309_5609_amd", "csrc"),
                    os.path.join(ROOT, "tests", "workspace_check.cpp"), "-o", str(exe)], check=True)

    def run(what):
        return subprocess.run([str(exe), what], capture_output=True, text=True).stdout.strip()

    return run


def test_a_captured_calls_buffers_stay(check):
    """What a call under capture was given is neither freed nor moved by longer calls after it."""
    assert check("graph") == "ok"


def test_memory_is_given_back_when_it_runs_out(check):
    """Buffers of earlier calls make room; those of the present call, and those in a graph, stay."""
    assert check("give_back") == "ok"
