"""The list rebuild's run of entries and row masks, built for the host: optimised, where a compiler uses
what the language leaves undefined, and with the undefined-behaviour sanitizer."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2109_11001_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("flags", [["-O3"], ["-O1", "-fsanitize=undefined", "-fno-sanitize-recover=undefined"]])
def test_list_run_on_the_host(tmp_path, flags):
    exe = str(tmp_path / "list_run")
    subprocess.run(["g++", "-std=c++17", *flags, "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I" + CSRC, os.path.join(HERE, "list_run_main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
