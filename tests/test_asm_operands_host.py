"""The broadcast FMAs written as assembly blocks of four: the compiler must not
give an input that a later instruction of the block reads the register of an
earlier instruction's result, whatever values the operands share.  Compiled for
gfx950 on the host, with equal values in results and inputs, and checked in the
assembly."""

import os
import re
import subprocess

import pytest

from paper_2301_05844_amd import build

FUNCTIONS = ("dot_bcast", "fma_bcast4", "axpy_bcast")
KERNELS = {
    # p[0] and the second input hold one value
    "dot_bcast": "double p[4] = {y, 1.0, 2.0, 3.0}; v4d t = {x[64], y, x[65], x[66]};"
                 "dot_bcast<3>(p, t);",
    # x[0] and the broadcast input
    "fma_bcast4": "double p[4] = {y, 1.0, 2.0, 3.0};"
                  "fma_bcast4<0>(p, x[64], x[65], x[66], x[67], y);",
    # x[0] and the coefficient
    "axpy_bcast": "v4d p = {y, 1.0, 2.0, 3.0}; axpy_bcast<0>(p, y);",
}


def _function(text, name):
    start = text.rindex("template <int", 0, text.index(f"void {name}("))
    return text[start:text.index("\n}\n", start) + 3]


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    with open(os.path.join(build.CSRC, "bbp_kernels.hip")) as f:
        text = f.read()
    src = ("#include <hip/hip_runtime.h>\n"
           "typedef double v4d __attribute__((ext_vector_type(4)));\n")
    src += "".join(_function(text, n) for n in FUNCTIONS)
    for n in FUNCTIONS:
        src += (f'extern "C" __global__ void k_{n}(double *o, const double *x) {{'
                f"double y = x[threadIdx.x]; {KERNELS[n]}"
                "for (int i = 0; i < 4; ++i) o[i * 64 + threadIdx.x] = p[i]; }\n")
    d = tmp_path_factory.mktemp("asm")
    hip, out = str(d / "k.hip"), str(d / "k.out")
    with open(hip, "w") as f:
        f.write(src)
    flags = [f for f in build.HIPCC_FLAGS if f != "-fPIC"]
    subprocess.run([build.hipcc(), *flags, "--cuda-device-only", "-S", hip, "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        text = f.read()
    got = {}
    for n in FUNCTIONS:
        body = text[text.index(f"\nk_{n}:"):]
        got[n] = re.search(r"ASMSTART\n(.*?)ASMEND", body, re.S).group(1)
    return got


@pytest.mark.parametrize("name", FUNCTIONS)
def test_no_input_in_an_earlier_result(blocks, name):
    fmacs = [re.findall(r"v\[(\d+):\d+\]", line) for line in blocks[name].splitlines()
             if "v_fmac_f64_dpp" in line]
    assert len(fmacs) == 4
    for i, (result, _, _) in enumerate(fmacs):
        for _, a, b in fmacs[i + 1:]:
            assert result not in (a, b), blocks[name]
