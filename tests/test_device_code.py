"""The one-wave coarsest solve passes its vector between lanes through LDS: its accesses have
to be LDS instructions, which a wave makes in order.  Compiled here with the library's flags and
looked at in the assembly; a pointer the compiler cannot place makes generic (flat) accesses."""
import re
import subprocess

import pytest

from paper_2501_13046_amd import build

SOURCE = """
#include "mg_bottom.hpp"
namespace grtmg {
template __global__ void k_bottom_psi<kBcPeriodic, float>(const BottomArgs<float>);
template __global__ void k_bottom_psi<kBcRobin, float>(const BottomArgs<float>);
template __global__ void k_bottom_psi<kBcZero, double>(const BottomArgs<double>);
template __global__ void k_coarse_psi<kBcPeriodic, double>(Geo, int, const double *, const double *, double *, double *);
template __global__ void k_coarse_psi<kBcRobin, float>(Geo, int, const float *, const float *, float *, double *);
template __global__ void k_coarse_psi_block<kBcRobin, double, 1>(Geo, int, const double *, const double *, double *,
                                                                 double *);
template __global__ void k_coarse_psi_block<kBcZero, double, 1>(Geo, int, const double *, const double *, double *,
                                                                double *);
}
"""


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    d = tmp_path_factory.mktemp("asm")
    src, asm = d / "coarse.hip", d / "coarse.s"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", f"{build.ROOT}/include", "-I", f"{build.PKG}/csrc",
                    "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True, capture_output=True)
    text = asm.read_text()
    return {m.group(1): m.group(0)
            for m in re.finditer(r"^(_ZN5grtmg\S+):.*?^\s*\.end_amdhsa_kernel", text, re.M | re.S)
            if re.search("k_bottom_psi|k_coarse_psi", m.group(1))}


def test_coarsest_solve_addresses_lds(kernels):
    assert len(kernels) == 7
    for name, body in kernels.items():
        assert len(re.findall(r"^\s*ds_(read|load)", body, re.M)) > 0, name
        generic = re.findall(r"^\s*flat_(?:load|store|atomic)\S*", body, re.M)
        assert not generic, (name, len(generic))


def test_block_solve_keeps_its_vectors_in_registers(kernels):
    """One cell a thread (up to 1024 cells): taps and Krylov vectors without scratch memory."""
    for name, body in kernels.items():
        if "k_coarse_psi_block" in name:
            assert re.search(r"private_segment_fixed_size 0\b", body), name
