"""The generated device code of the scan kernels, built with the flags of the
library's units, has no lost copies.

A register copy that the compiler finds to be between the same register and
itself is left in the listing as a comment, `kill: def A killed A`.  With
vectorised FP32 code this compiler marked copies between different registers
the same way, so the value was never moved: the listing shows `kill: def B
killed A` with B and A apart.
"""
import os
import re
import subprocess

import pytest

from paper_2102_00514_amd import build

SOURCE = """
#include "operators.hpp"
#include "sqrt.hpp"
#include "scan.hpp"
namespace pks {
#define SCANS(OP, N, R)                                                        \\
  template __global__ void k_scan_up<OP<N, R, true>, 64, R>(ScanArgs);         \\
  template __global__ void k_scan_down<OP<N, R, true>, 64, R>(ScanArgs);       \\
  template __global__ void k_scan_single<OP<N, R, true>, 64, R>(ScanArgs);     \\
  template __global__ void k_scan_single<OP<N, R, true>, 256, R>(ScanArgs);
#define ALL(N, R) SCANS(FilterOp, N, R) SCANS(SmootherOp, N, R) SCANS(SqrtFilterOp, N, R) SCANS(SqrtSmootherOp, N, R)
ALL(5, REAL) ALL(3, REAL)
}
"""


def lost_copies(listing: str):
    out = []
    for d, s in re.findall(r"kill: def (\$\S+) killed (\$\S+)", listing):
        if not set(re.findall(r"[a-z]gpr\d+", d)) & set(re.findall(r"[a-z]gpr\d+", s)):
            out.append((d, s))
    return out


def listing(tmp_path, real, flags):
    src = tmp_path / "scans.hip"
    src.write_text(SOURCE.replace("REAL", real))
    dst = tmp_path / "scans.s"
    subprocess.run([build.HIPCC, *flags, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"),
                    "--cuda-device-only", "-S", "-o", str(dst), str(src)], check=True, capture_output=True, timeout=600)
    return dst.read_text()


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc is not available")
@pytest.mark.parametrize("unit", ["engine_ct_f32.hip", "engine_ct_f64.hip"])
def test_scan_kernels_have_no_lost_copies(tmp_path, unit):
    assert unit in build.UNITS
    assert all(build.unit_flags(u) == build.unit_flags(unit) for u in build.UNITS if u[-8:] == unit[-8:])
    text = listing(tmp_path, "float" if "_f32" in unit else "double", build.unit_flags(unit))
    assert text.count(".amdhsa_kernel ") == 32
    assert lost_copies(text) == []


def test_the_search_finds_one():
    assert lost_copies("; kill: def $vgpr23 killed $vgpr16 killed $exec\n"
                       "; kill: def $vgpr2 killed $vgpr2 killed $vgpr2_vgpr3 killed $exec\n") == [("$vgpr23", "$vgpr16")]
