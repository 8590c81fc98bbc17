"""The build without a compiler run: what is left out where a tool is missing, and what is not."""
import os
import re
import subprocess
import sys

import pytest

from paper_2407_16207_amd import build


@pytest.mark.parametrize("missing", ["nothing", "torch", "compiler", "headers"])
def test_the_library_is_built_where_the_native_binding_cannot_be(monkeypatch, tmp_path, capsys, missing):
    """The library needs hipcc alone; without torch, a host compiler or Python's headers the binding's native part is left out,
    with one line that says so and nothing left over from an earlier build."""
    binding, ran = tmp_path / "binding.so", []
    binding.write_text("of an earlier build")

    def check_call(cmd):
        ran.append(cmd)
        if str(binding) in cmd:
            assert missing != "torch"
            if missing == "compiler":
                raise FileNotFoundError(2, "No such file or directory", cmd[0])
            if missing == "headers":
                raise subprocess.CalledProcessError(1, cmd)
            binding.write_text("of this build")
    monkeypatch.setattr(build, "BINDING_PATH", str(binding))
    monkeypatch.setattr(build.subprocess, "check_call", check_call)
    if missing == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)
    assert build.build_library() == build.LIB_PATH
    outputs = [cmd[cmd.index("-o") + 1] for cmd in ran]
    assert build.LIB_PATH in outputs and build.BENCH_LIB_PATH in outputs
    said = capsys.readouterr().out.splitlines()
    if missing == "nothing":
        assert binding.read_text() == "of this build" and not said
    else:
        assert not binding.exists() and len(said) == 1 and "binding.so was not built" in said[0]


def test_a_library_that_does_not_compile_is_an_error(monkeypatch):
    def check_call(cmd):
        raise subprocess.CalledProcessError(1, cmd)
    monkeypatch.setattr(build.subprocess, "check_call", check_call)
    with pytest.raises(subprocess.CalledProcessError):
        build.build_library()


def kernels_of(path, workdir):
    """Per kernel in a library built here: what the compiler notes about it."""
    readelf = "/opt/rocm/llvm/bin/llvm-readelf"
    if not os.path.exists(path) or not os.path.exists(readelf):
        pytest.skip("needs the built library and ROCm's llvm-readelf")
    image = open(path, "rb").read()
    starts = [m.start() for m in re.finditer(b"\x7fELF", image)][1:]           # the first is the library itself
    found = {}
    for lo, hi in zip(starts, starts[1:] + [len(image)]):
        (workdir / "object").write_bytes(image[lo:hi])
        notes = subprocess.run([readelf, "--notes", str(workdir / "object")], capture_output=True, text=True).stdout
        for entry in notes.split(".agpr_count:")[1:]:
            found[re.search(r"\.name: +(_Z\S+)", entry)[1]] = {k: int(v) for k, v in re.findall(r"\.(\w+): +(\d+)\n", entry)}
    return found


def test_sampling_kernels_do_not_spill_registers(tmp_path):
    """The general draw's scan once kept sixteen 64-bit lane masks at a time: 30 scalar registers went to lanes of vector
    registers and back, which cost calls of more than 256 sequences up to 5 %."""
    kernels = {name: k for name, k in kernels_of(build.LIB_PATH, tmp_path).items() if "resample" in name or "accept" in name}
    assert len(kernels) >= 9
    assert not {name: k for name, k in kernels.items() if k["sgpr_spill_count"] or k["vgpr_spill_count"]}
