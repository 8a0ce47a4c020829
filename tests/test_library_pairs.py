"""Pair arithmetic of the operator tables: compiled for the host, against exact
rationals; compiled for the device with the library's flags, the operations of
one sum and product, none of them contracted.

Tolerance: s + a b on pairs of 53-bit numbers loses a few units of 2^-106 of
its largest term; 2^-100 of |s| + |a b| leaves room for eight of the
operations, and a product whose rounding error is lost or counted twice is off
by up to 2^-53 of it.
"""
import ctypes
import os
import re
import subprocess
from fractions import Fraction

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1705_03838_amd", "csrc")
SOURCE = """
#include "opf_pair.h"
extern "C" void madds(int n, const double* s, const double* a, const double* b, double* out) {
    for (int i = 0; i < n; ++i) {
        const opf::dd r = madd(opf::dd{s[2 * i], s[2 * i + 1]}, opf::dd{a[2 * i], a[2 * i + 1]}, b[i]);
        out[2 * i] = r.hi;
        out[2 * i + 1] = r.lo;
    }
}
"""


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
@pytest.mark.skipif("fma" not in open("/proc/cpuinfo").read(), reason="needs a processor with multiply-add")
def test_sum_and_product_of_pairs(tmp_path):
    src, lib = tmp_path / "pairs.hip", tmp_path / "pairs.so"
    src.write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xarch_host", "-mfma", "-fPIC",
                    "-shared", "-w", "-I", CSRC, str(src), "-o", str(lib)], check=True, timeout=300)
    rng = np.random.default_rng(1)
    n = 4000
    s, a = (np.empty((n, 2)) for _ in range(2))
    for x in (s, a):
        x[:, 0] = rng.standard_normal(n) * 2.0 ** rng.integers(-20, 20, n)
        x[:, 1] = x[:, 0] * rng.uniform(-1, 1, n) * 2.0 ** -54
    b = rng.standard_normal(n)
    s[:400, 0] = -a[:400, 0] * b[:400]  # the sum cancels but for the product's rounding error
    s[:400, 1] = 0.0
    out = np.empty((n, 2))
    p = ctypes.POINTER(ctypes.c_double)
    ctypes.CDLL(str(lib)).madds(n, *(v.ctypes.data_as(p) for v in (s, a, b, out)))
    worst = 0.0
    for i in range(n):
        S, A, B, R = (Fraction(float(v[0])) + Fraction(float(v[1])) for v in (s[i], a[i], (b[i], 0.0), out[i]))
        worst = max(worst, float(abs(R - (S + A * B)) / (abs(S) + abs(A * B))))
    assert worst <= 2.0 ** -100, worst


KERNEL = """
#include "opf_pair.h"
extern "C" __global__ void product(const opf::dd* a, const double* b, opf::dd* out) { *out = madd(*out, *a, *b); }
"""


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_device_product_is_not_contracted(tmp_path):
    from paper_1705_03838_amd.build import FLAGS, HIPCC
    src, out = tmp_path / "product.hip", tmp_path / "product.s"
    src.write_text(KERNEL)
    flags = [f for f in FLAGS if f != "-fPIC"]
    subprocess.run([HIPCC, *flags, "-w", "--cuda-device-only", "-S", "-I", CSRC, str(src), "-o", str(out)], check=True,
                   timeout=300)
    ops = re.findall(r"^\s+v_(mul|fma|fmac|add)_f64", out.read_text(), re.M)
    # a_hi b; its error and a_lo b to it; the sum with its error (six) and the low parts (two)
    assert (ops.count("mul"), ops.count("fma") + ops.count("fmac"), ops.count("add")) == (1, 2, 8), ops
