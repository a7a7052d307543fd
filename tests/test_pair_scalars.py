"""The FP64 pair kernels' point arithmetic (kappa64.h, ssq_map.h), compiled for
the host, against long double: closed-form kernel differences from a root and
an inverse root without divisions, and the P2 polynomials of the singular pairs.

The yardstick is the same quantity by its definition in double.  Both round a
few dozen times; 10 % is more than 200 000 points (0.2 %) and the order of the
operations account for.  The polynomials have fewer operations than the sum
over six nodes and smaller terms, so they are held to the sum's own error."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pair_scalars") / "pair_scalars")
    # contraction as in the device code; w: HIP's headers outside hipcc
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-mfma", "-ffp-contract=fast", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-I" + os.path.join(ROCM, "include"), os.path.join(HERE, "pair_scalars.cpp"), "-o", exe])

    def run(*args):
        out = subprocess.check_output([exe, *map(str, args)], text=True)
        return {name: (float(got), float(yard)) for name, got, yard in map(str.split, out.splitlines())}
    return run


@pytest.mark.parametrize("k0,eps", [(1.0, 4.0), (1.3, 3.0 + 0.1j), (5.0, 2.25), (3.0, -10.0 + 1.5j)])
def test_closed_forms_are_as_accurate_as_their_definitions(driver, k0, eps):
    for name, (got, yard) in driver(k0, eps.real, complex(eps).imag).items():
        assert got <= 1.1 * yard, (name, got, yard)


def test_polynomials_are_as_accurate_as_nodal_sums(driver):
    got, yard = driver()["p2"]
    assert got <= yard
