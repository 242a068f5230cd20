"""The formats the kernels on float32 values can be generated for: the arithmetic's
conditions hold for every variant of the table (the build compiles them) and refuse,
when compiled, formats it is not exact for."""
import os
import subprocess

import pytest

from paper_2007_06563_amd import build, variants

SRC = """
#include "value.hpp"
struct V {{
  static constexpr int NIN = {nin}, NACC = {nacc}, NOUT = {nacc};
  static constexpr int wE = {wE}, wF_IN = {wi}, wF_ACC = {wa}, wF_OUT = {wa};
  static constexpr int kAct = 0, kRound = {rnd};
}};
{what}
"""
CONV = ("hipError_t f(const hobflops::ConvParams& p) "
        "{ return hobflops::launch_value<V>(nullptr, nullptr, nullptr, p, 0, nullptr); }")
POOL = "template __global__ void hobflops::avgpool_value_kernel<V>(const uint32_t*, uint32_t*, hobflops::PoolParams);"


@pytest.mark.parametrize("fmt,what,ok", [
    ((6, 4, 5, 0), CONV, True),    # a wider exponent than the table's
    ((7, 4, 5, 0), CONV, False),   # scaled products leave float32's range
    ((8, 7, 8, 0), CONV, False),
    ((5, 11, 12, 0), CONV, False),  # products of 24 bits, to nearest
    ((5, 10, 23, 0), CONV, False),  # no bit of float32 left to round at
    ((5, 11, 11, 0), POOL, True),
    ((5, 12, 12, 0), POOL, False),  # the product with the scale has 26 bits
], ids=str)
def test_conditions_of_the_arithmetic(tmp_path, fmt, what, ok):
    wE, wi, wa, rnd = fmt
    src = tmp_path / "v.hip"
    src.write_text(SRC.format(nin=3 + wE + wi, nacc=3 + wE + wa, wE=wE, wi=wi, wa=wa, rnd=rnd,
                              what=what))
    r = subprocess.run([build.HIPCC, "-fsyntax-only", "--offload-arch=gfx950", "-std=c++17", "-I",
                        os.path.join(build.HERE, "csrc"), str(src)],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == ok, r.stderr[-2000:]
    assert ok or "static assertion failed" in r.stderr, r.stderr[-2000:]


@pytest.mark.parametrize("fmt,ops", [
    ((5, 3, 4, variants.RNE), 7), ((5, 9, 10, variants.RNE), 8), ((5, 3, 7, variants.RNE), 5),
    ((5, 10, 11, variants.RNE), 16), ((5, 10, 21, variants.RNE), 13), ((5, 3, 4, variants.RTZ), 4),
    ((5, 3, 7, variants.RTZ), 3),
    ((4, 9, 10, variants.RNE), 7),  # a bias of 7: products need no scaling back
], ids=str)
def test_operation_counts(fmt, ops):
    """The count that AUTO's estimate and the benchmark's bound use, by hand: product
    1; its rounding 2, scaled back 1 more where 2^(23 - wF) is below 2^bias; a sum and
    its rounding 4, in float64 six of two each; toward zero 1 for each step."""
    assert build.value_ops(*fmt) == ops
