"""The division of an attention call's query tiles between kernels, checked on
the host: every tile is in exactly one part, and no call takes more rounds of the
chip than the same tiles in the plain form of 128-query workgroups."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_02584_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text('#include "ra_plan.h"\n'
                   'extern "C" void fallback(int npad, int bh, int kv, int units, int* o) {\n'
                   '  const ra::TilePlan p = ra::plan_fallback(npad, bh, kv, units);\n'
                   '  o[0] = p.whole, o[1] = p.halves, o[2] = p.quarters, o[3] = p.tiles128;\n}\n'
                   'extern "C" void e2m3(int npad, int bh, int kv, int ktok, int units, int* o) {\n'
                   '  const ra::TilePlan p = ra::plan_e2m3(npad, bh, kv, ktok, units);\n'
                   '  o[0] = p.whole, o[1] = p.halves, o[2] = p.quarters, o[3] = p.tiles128;\n}\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))

    def call(name, *args):
        o = (ctypes.c_int * 4)()
        getattr(lib, name)(*args, o)
        return tuple(o)
    return call


# a whole chip, partitions of it, and a number that the fractions do not divide
UNITS = [256, 128, 64, 32, 38]


@pytest.mark.parametrize("units", UNITS)
@pytest.mark.parametrize("kv", [64, 128])
def test_fallback_plan(plan, kv, units):
    for n128 in (1, 2, 3, 4, 5, 7, 9, 12, 13, 33, 256):
        for bh in list(range(1, 600)) + [640, 1000, 4096]:
            whole, halves, quarters, tiles128 = plan("fallback", 128 * n128, bh, kv, units)
            total = -(-n128 // 2) * bh
            if tiles128:
                assert (whole, halves, quarters) == (0, 0, 0) and tiles128 == n128 * bh and kv == 64
            else:
                assert whole + halves + quarters == total and not (halves and quarters)
                assert 2 * halves <= units and 4 * quarters <= units
            # rounds: 256-query workgroups one a unit, 128-query ones two (kv_block 64)
            rounds = -(-whole // units) + (halves + quarters > 0) + -(-tiles128 // (2 * units))
            if kv == 64:
                assert rounds <= -(-(n128 * bh) // (2 * units)), (n128, bh)


@pytest.mark.parametrize("units", UNITS)
@pytest.mark.parametrize("kv,ktok", [(64, 0), (64, 1), (128, 0), (128, 1)])
def test_e2m3_plan(plan, kv, ktok, units):
    """Whole rounds on the 8-wave kernel, and a last round of at most half the
    units in smaller workgroups, one a unit (quarters of per-token scales: two)."""
    for total in range(1, 4 * units):
        whole, halves, quarters, tiles128 = plan("e2m3", 256, total, kv, ktok, units)
        assert whole + halves + quarters == total and not tiles128 and not (halves and quarters)
        rest = total % units
        assert halves + quarters == (rest if 2 * rest <= units else 0)
        assert 2 * halves <= units and 4 * quarters <= (2 if ktok else 1) * units
        assert not quarters or kv == 128
        assert not halves or kv == 64 or not ktok     # the kernels that are built
