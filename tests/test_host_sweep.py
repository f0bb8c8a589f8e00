"""The 16-row sweep's loads and stores, walked on the CPU: no address outside the caller's matrices is formed, whatever a
buffer's bounds check makes of the row's offset."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def reach(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("reach") / "reach")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([os.path.join(rocm, "llvm", "bin", "clang++"), "-std=c++17", "-O1", "-w", "-o", exe, os.path.join(HERE, "sweep16_reach.cpp")],
                   check=True, timeout=120)
    return exe


# fewer columns than a super-block, a last one of 4 columns to one short of full, rows that end inside a workgroup, far runs of every kind
@pytest.mark.parametrize("beta1", [4, 8, 16, 32])
def test_no_address_outside_the_matrices(reach, beta1):
    sizes = [(m, n) for m in (2, 16, 18, 32) for n in (beta1, 64, 96, 128, 128 + beta1, 256, 256 + beta1, 384 - beta1, 384 + beta1, 512 + 2 * beta1, 1120)]
    got = subprocess.run([reach] + [str(v) for m, n in sizes + [(20, 2720)] for v in (beta1, m, n)], capture_output=True, text=True, timeout=120)
    assert got.returncode == 0, got.stdout.splitlines()[-1]
    assert len(got.stdout.splitlines()) == len(sizes) + 1


# layers of which either kernel was measured to be faster by a tenth or more: rows, columns, beta1, outlier tests, rows of the faster one
@pytest.mark.parametrize("m,n,b1,tests,rows", [
    (4096, 64, 4, 0, 16), (8192, 64, 4, 0, 64), (8192, 256, 4, 0, 16), (12288, 256, 4, 0, 64), (12288, 256, 4, 1, 64), (8192, 512, 4, 1, 16),
    (16384, 1024, 4, 1, 64), (20480, 1024, 4, 1, 16), (32768, 2048, 4, 0, 16), (16384, 512, 8, 0, 64), (12288, 64, 8, 0, 64), (12288, 64, 8, 1, 16),
    (16384, 1024, 8, 0, 16), (16384, 256, 16, 0, 64), (16384, 256, 16, 1, 16), (8192, 64, 16, 0, 16), (12288, 512, 16, 0, 16),
    (32768, 256, 32, 0, 64), (65536, 512, 32, 0, 64), (65536, 512, 32, 1, 16), (16384, 2048, 32, 0, 16), (11008, 4096, 16, 0, 16)])
def test_rows_a_workgroup(m, n, b1, tests, rows):
    import ctypes
    import paper_2306_03078_amd as P
    lib = ctypes.CDLL(P.library_path())
    assert lib.spqr_sweep_rows(m, n, b1, 16, tests) == rows
    assert lib.spqr_sweep_rows(m, n, b1, 32, tests) == 64           # tiles of more than 16 rows
