"""What the build asks of the machine it runs on."""
import importlib.util
import os
import re
import shutil
import subprocess
import sys

import pytest

from paper_2503_22879_amd import build


@pytest.mark.parametrize("how", ["path", "link", "full"])
def test_hip_headers_beside_a_compiler_that_path_or_a_link_finds(monkeypatch, tmp_path, how):
    full = shutil.which(build.HIPCC) or build.HIPCC
    if how == "path":
        monkeypatch.setenv("PATH", os.path.dirname(full) + os.pathsep + os.environ["PATH"])
        monkeypatch.setattr(build, "HIPCC", os.path.basename(full))
    elif how == "link":
        os.symlink(full, tmp_path / "cc")
        monkeypatch.setattr(build, "HIPCC", str(tmp_path / "cc"))
    monkeypatch.setattr(build, "BIND", str(tmp_path / "_bind.so"))
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    ran = []
    monkeypatch.setattr(build.subprocess, "check_call", ran.append)
    build._build_bind(True)
    found = [d for flag, d in zip(ran[0], ran[0][1:]) if flag == "-isystem" and
             os.path.exists(os.path.join(d, "hip", "hip_runtime.h"))]
    assert found and all(os.path.isabs(d) for d in found)


def test_the_c_library_is_built_where_the_extension_cannot_be(monkeypatch, tmp_path):
    """Without torch, and with a compiler for the extension that fails."""
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "_compile", lambda src, force: src + ".o")
    ran = []

    def check_call(cmd):
        ran.append(cmd)
        if build.BIND in cmd:
            raise FileNotFoundError(cmd[0])

    monkeypatch.setattr(build.subprocess, "check_call", check_call)
    with pytest.raises(FileNotFoundError):
        build.build_library()
    assert any(build.LIB in cmd for cmd in ran)
    ran.clear()
    monkeypatch.setitem(sys.modules, "torch", None)
    monkeypatch.setattr(importlib.util, "find_spec", lambda name: None)
    assert build.build_library() == build.LIB
    assert len(ran) == 1 and build.LIB in ran[0]


def test_the_extension_is_built_again_for_another_torch(monkeypatch, tmp_path):
    import torch
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "BIND", str(tmp_path / "_bind.so"))
    ran = []

    def check_call(cmd):
        ran.append(cmd)
        open(build.BIND, "w").close()

    monkeypatch.setattr(build.subprocess, "check_call", check_call)
    for _ in range(2):
        build._build_bind(False)
    assert len(ran) == 1
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".other")
    for _ in range(2):
        build._build_bind(False)
    assert len(ran) == 2


@pytest.mark.parametrize("source,kernel", [("mamba1.hip", "mamba1_scan_halves_kernel"), ("prefill_wide.hip", "prefill_wide_kernel")])
def test_kernels_that_fill_their_registers_keep_everything_in_them(tmp_path, source, kernel):
    """By the compiler's report: no scratch memory in the kernels whose waves have 128 registers and several bodies to fit into them."""
    cmd = [build.HIPCC, *build.FLAGS, "-x", "hip", "--cuda-device-only", "-c", os.path.join(build.CSRC, source), "-o",
           str(tmp_path / "o"), "-Rpass-analysis=kernel-resource-usage"]
    report = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    scratch = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", report, re.S)
    found = {name: int(size) for name, size in scratch if kernel in name}
    assert found and not any(found.values()), found
