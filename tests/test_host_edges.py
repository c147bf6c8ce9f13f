"""The library's host code at the edges, on the CPU: calls made while a stream captures, and runtime calls that fail.

The library's sources are compiled for the host only and linked against the stand-in for the HIP runtime
(hostcheck/hip_stub.cpp; kernels do nothing, and what HIP forbids under capture is an error) and hostcheck/edges.cpp,
whose wrappers make runtime calls fail on demand.
"""
import concurrent.futures
import os
import subprocess

import numpy as np
import pytest

from paper_1307_3218_amd import lattice

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1307_3218_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.path.join(ROCM, "bin", "hipcc")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")
WRAPPED = ["hipStreamSynchronize", "hipMalloc", "hipFree", "hipMemGetInfo"]


def _compile(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{' '.join(cmd)}\n{r.stdout[-3000:]}\n{r.stderr[-3000:]}")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not (os.path.exists(HIPCC) and os.path.exists(CLANG)):
        pytest.skip("hipcc / clang++ of the ROCm toolchain not found")
    tmp = tmp_path_factory.mktemp("edges")
    lib = ["-O0", "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-w", '-DMAR_BUILD_ID="edges"']
    host = ["-O0", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", os.path.join(ROCM, "include"), "-I",
            os.path.join(ROOT, "include")]
    jobs = []
    for f in sorted(os.listdir(CSRC)):
        if f.endswith((".hip", ".cpp")):
            jobs.append([HIPCC] + lib + (["-x", "hip"] if f.endswith(".hip") else []) +
                        ["-c", os.path.join(CSRC, f), "-o", str(tmp / (f + ".o"))])
    for f in ("hip_stub.cpp", "edges.cpp"):
        jobs.append([CLANG] + host + ["-c", os.path.join(HERE, "hostcheck", f), "-o", str(tmp / (f + ".o"))])
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        list(ex.map(_compile, jobs))
    exe = str(tmp / "edges")
    _compile([CLANG, "-o", exe] + sorted(str(tmp / f) for f in os.listdir(tmp) if f.endswith(".o")) +
             [f"-Wl,--wrap={w}" for w in WRAPPED] + ["-lpthread", "-Wl,--unresolved-symbols=ignore-in-object-files"])
    s = lattice.generate(4, 4, 2, seed=0)
    H, S = s.H.tocsr(), s.S.tocsr()
    with open(tmp / "sys.bin", "wb") as f:
        np.array([s.M, H.nnz, S.nnz], dtype=np.int64).tofile(f)
        for A in (H, S):
            A.indptr.astype(np.int64).tofile(f)
            A.indices.astype(np.int32).tofile(f)
            A.data.astype(np.float64).tofile(f)
    return exe, str(tmp / "sys.bin")


def _run(program, scenario, *args):
    r = subprocess.run([program[0], scenario, program[1], *map(str, args)], capture_output=True, text=True, timeout=120)
    out = r.stdout + r.stderr
    print(out)
    assert r.returncode == 0 and "stub errors 0" in out, out
    return out


def test_local_region_set_while_a_stream_captures(program):
    assert "status 0 hops 3" in _run(program, "region_under_capture")


def test_failing_measurement_of_the_regions_is_reported(program):
    out = _run(program, "region_sizes_fail")
    assert "setter 0, solve -5 (hipStreamSynchronize" in out and "again 0" in out


def test_more_seeds_under_capture_than_in_the_warm_call(program):
    assert _run(program, "more_seeds_under_capture").count("warm 0, captured 0") == 4


def test_basis_of_an_eigen_state_gives_way_to_a_later_solve(program):
    assert "eigen state 0, tuning 0, solve 0" in _run(program, "kept_basis_gives_way")


def test_eigen_state_without_room_for_the_pass_beside_the_kept_basis(program):
    assert "eigen state 0, on less memory 0" in _run(program, "kept_basis_without_room_for_the_pass")


@pytest.mark.parametrize("form,warm,captured", [
    ("seeds", 130, 200), ("seeds", 300, 1024), ("blocks", 64, 100), ("blocks", 128, 255), ("blocks", 512, 300),
    ("blocks", 256, 300), ("blocks", 256, 290), ("blocks", 1024, 140), ("textbook", 64, 100),
    ("then_blocks", 200, 100), ("then_blocks", 130, 1024), ("then_region", 200, 100), ("then_region", 130, 20)])
def test_another_number_of_seeds_under_capture(program, form, warm, captured):
    """Counts that take the same block width or fewer than before, and a captured call in seed blocks after a warm one of
    one workgroup per seed (then_*): the captured call runs in the workspace of the warm one."""
    assert _run(program, "seed_counts_under_capture", warm, captured, form).count("warm 0, captured 0") == 2
