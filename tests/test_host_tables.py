"""The tables that the library's host code builds for the banded and the sparse step, read back as
the kernels read them (tests/host_tables.cpp, compiled here from that code alone, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1911_08801_amd", "csrc")
DTYPES = {"f32": 0, "bf16": 1, "f16": 2}


@pytest.fixture(scope="module")
def tables(tmp_path_factory):
    cc = shutil.which("g++") or "/opt/rocm/llvm/bin/clang++"
    exe = str(tmp_path_factory.mktemp("host") / "host_tables")
    subprocess.run([cc, "-O2", "-std=c++17", "-I", CSRC, "-o", exe, os.path.join(ROOT, "tests", "host_tables.cpp"),
                    os.path.join(CSRC, "asn_host.cpp")], check=True)

    def run(*args):
        r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0
        return r.stdout
    return run


# (n_polar, n_azim, operand type, beta): reach 0 to 3, narrow runs, whole rings, both ends of the
# azimuth counts, one level
BANDED = [(1, 8, "f32", 4.5), (2, 8, "f32", 2.0), (4, 8, "f32", 40.0), (8, 16, "f32", 4.5), (4, 16, "f32", 13.0),
          (12, 24, "f32", 9.0), (3, 56, "f32", 4.5), (4, 64, "f32", 40.0), (2, 32, "bf16", 9.0), (4, 32, "f16", 40.0),
          (16, 32, "bf16", 9.0), (4, 48, "bf16", 20.0), (4, 48, "f16", 200.0), (4, 64, "bf16", 20.0),
          (8, 64, "f16", 13.0)]


@pytest.mark.parametrize("n_polar,n_azim,dtype,beta", BANDED)
def test_row_defect_of_the_coefficients_multiplied(tables, n_polar, n_azim, dtype, beta):
    # c(-d) one number of the operand type above c(d), of which the kernel multiplies the latter
    assert tables("defect", n_polar, n_azim, DTYPES[dtype], beta) == ""


@pytest.mark.parametrize("n_polar,n_azim,dtype,beta", BANDED)
def test_banded_tables_give_the_stored_kernel_back(tables, n_polar, n_azim, dtype, beta):
    # from each reach's table, by its offsets, flags and step counts, +-d one coefficient
    assert tables("band", n_polar, n_azim, DTYPES[dtype], beta) == ""


# (n_polar, n_azim, icosahedron order, operand type, beta): ordinates that fill the last group or
# not, and the last 64-ordinate word or not; a sparse and a dense K
SPARSE = [(1, 2, 0, "f32", 4.5), (5, 10, 0, "bf16", 4.5), (8, 16, 0, "f16", 9.0), (1, 4, 2, "f32", 4.5),
          (1, 4, 3, "f16", 4.5), (1, 4, 5, "f32", 4.5), (1, 4, 5, "f32", 80.0), (1, 4, 7, "bf16", 4.5)]


@pytest.mark.parametrize("n_polar,n_azim,ico,dtype,beta", SPARSE)
def test_sparse_tables_give_the_stored_kernel_back(tables, n_polar, n_azim, ico, dtype, beta):
    assert tables("sparse", n_polar, n_azim, ico, DTYPES[dtype], beta, 4, 8) == ""
