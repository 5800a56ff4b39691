"""The on-chip preconditioner's waits, marks and barriers (resident.hip), shown on the
CPU: the kernel's own source runs as fibers, one wavefront at a time, in orders that a
GPU takes only now and then (emulation/onchip_emulation.cpp)."""

from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_17850_amd", "csrc")
CLANG = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)


def _host_source(name):
    """A kernel file with what only the device compiler takes replaced."""
    text = open(os.path.join(CSRC, name)).read()
    text = text.replace('asm volatile("v_mov_b32 %0, %1" : "=v"(c) : "v"(w[i]));', "c = w[i];")
    text = re.sub(r'asm volatile\("" :[^;]*\);', "", text)
    text = text.replace("extern __shared__ __align__(16) unsigned char lds_raw[];",
                        "unsigned char *lds_raw = emu::dynamic_lds();")
    text = re.sub(r"__attribute__\(\(address_space\(\d\)\)\)", "", text)
    text = text.replace("__shared__", "static thread_local")
    # (lanes run in lockstep: the edge corrections are written before they are read)
    text = text.replace("if (x_edge) {", "emu::cross(emu::kWave, 0, 0);\n        if (x_edge) {")
    return text


def _build(tmp, name, main, extra=""):
    """tests/emulation/<main> over the host form of the kernel sources."""
    for f in ("device_util.hpp", "resident.hip"):
        text = _host_source(f)
        if f == "resident.hip":
            f = "onchip_kernel.inc"
            text += extra
        with open(os.path.join(tmp, f), "w") as out:
            out.write(text)
    exe = os.path.join(tmp, name)
    subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-pthread", "-I", str(tmp), "-I", os.path.join(HERE, "emulation"),
                    "-I", CSRC, os.path.join(HERE, "emulation", main), "-o", exe], check=True)
    return exe


@pytest.fixture(scope="module")
def emulation(tmp_path_factory):
    if CLANG is None:
        pytest.skip("no clang")
    return _build(tmp_path_factory.mktemp("onchip"), "emulation", "onchip_emulation.cpp")


def _run(exe, scenario, seed):
    out = subprocess.run([exe, scenario, str(seed)], stdout=subprocess.PIPE, timeout=100, check=True)
    return out.stdout.decode().strip()


def test_units_of_a_device_are_shared(tmp_path):
    """Eight threads take 1 to all of the compute units: never more in all than there
    are, small ones together, and none waits for ever; a process ends while one waits."""
    if CLANG is None:
        pytest.skip("no clang")
    exe = str(tmp_path / "lease")
    subprocess.run([CLANG, "-std=c++17", "-O1", "-pthread", "-I", CSRC, os.path.join(HERE, "emulation", "lease.cpp"),
                    "-o", exe], check=True)
    for args in ([], ["exit"]):
        assert subprocess.run([exe, *args], stdout=subprocess.PIPE, timeout=30, check=True).stdout == b"ok\n"


@pytest.mark.parametrize("seed", range(4))
def test_sound_applications(emulation, seed):
    assert _run(emulation, "runs", seed) == "ok"


@pytest.mark.parametrize("seed", range(16))
def test_stop_flag_is_the_workgroups(emulation, seed):
    """The lead tile stores the stop flag of a converged problem while other tiles
    read it: all wavefronts of a workgroup act on one reading of it."""
    assert _run(emulation, "converged", seed) == "ok"


@pytest.mark.parametrize("seed", range(16))
def test_a_mark_parts_no_workgroup(emulation, seed):
    """A tile gives up while wavefronts of a neighbour start: they leave together, and
    the problem that the workgroups take next is sound."""
    assert _run(emulation, "gave_up", seed) == "ok"


@pytest.mark.parametrize("seed", range(4))
def test_late_lead_tile_counts_the_iteration(emulation, seed):
    """The solve goes on from the count of updates, also where the tile that counts
    them starts after another has given up."""
    assert _run(emulation, "late_lead", seed) == "ok"


def test_every_tile_shape_has_a_kernel(emulation):
    """The shapes that the host chooses from: 64 x 8 columns in every layer class (FP64:
    up to 16), in FP32 64 x 16 up to 16 layers and, plain per layer, 64 x 14 at 20."""
    built = _run(emulation, "shapes", 0).split()
    want = {"ok"}
    for cells in (0, 1):
        for jacobi in (0, 1):
            want |= {f"{nz}:{size}{cells}{jacobi}:1x8" for nz in (8, 12, 16, 20) for size in (4, 8) if nz <= 16 or size == 4}
            want |= {f"{nz}:4{cells}{jacobi}:2x8" for nz in (8, 12, 16)}
    assert want | {"20:400:2x7"} == set(built)
