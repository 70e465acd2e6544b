"""A plan whose step stopped between two launches (the launch's failure is forced by the host) steps correctly afterwards:
tests/native/stopped_step.c."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def compile_program(tmp_path):
    lib = os.environ.get("ECO_LIB_PATH") or os.path.join(ROOT, "paper_2601_22101_amd", "libeco.so")
    exe = str(tmp_path / "stopped_step")
    cmd = ["gcc", "-O1", "-std=gnu11", "-Wall", "-Wextra", "-Werror", "-Wno-unused-parameter", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "stopped_step.c"), "-o", exe, "-Wl,--export-dynamic",
           "-L", os.path.dirname(lib), "-l:" + os.path.basename(lib), "-L/opt/rocm/lib", "-lamdhip64", "-ldl",
           "-Wl,-rpath," + os.path.dirname(os.path.abspath(lib)), "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return exe


def test_the_program_compiles(tmp_path):
    from paper_2601_22101_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    compile_program(tmp_path)


@pytest.mark.gpu
def test_a_plan_steps_correctly_after_a_step_that_stopped_between_launches(tmp_path):
    r = subprocess.run([compile_program(tmp_path)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=100)
    assert r.returncode == 0 and "stopped step ok" in r.stdout, r.stdout[-3000:]
