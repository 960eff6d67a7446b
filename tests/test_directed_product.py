"""mul_down (sbr_common.h), the directed product of the slab test's offsets, is
at most the exact product, and not below it by more than two ulps.  The
function's own text is compiled for the host and called here."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def mul_down(tmp_path_factory):
    with open(os.path.join(ROOT, "paper_2504_21719_amd", "csrc", "sbr_common.h")) as f:
        body = re.search(r"float mul_down\(float a, float b\) \{\n.*?\n\}\n", f.read(), re.S).group(0)
    d = tmp_path_factory.mktemp("mul_down")
    src, so = str(d / "m.cpp"), str(d / "m.so")
    with open(src, "w") as f:
        f.write("#include <cmath>\nusing std::fabs;\nstatic inline %s"
                "extern \"C\" void run(const float* a, const float* b, float* c, long n) {"
                " for (long i = 0; i < n; i++) c[i] = mul_down(a[i], b[i]); }\n" % body)
    subprocess.check_call(["g++", "-O2", "-ffp-contract=off", "-shared", "-fPIC", src, "-o", so])
    run = C.CDLL(so).run
    run.argtypes = [C.c_void_p] * 3 + [C.c_long]

    def call(a, b):
        c = np.empty_like(a)
        run(a.ctypes.data, b.ctypes.data, c.ctypes.data, len(a))
        return c
    return call


def _check(call, a, b):
    a, b = a.astype(np.float32), b.astype(np.float32)
    c = call(a, b)
    exact = a.astype(np.float64) * b.astype(np.float64)          # 48 bits: exact
    assert np.all(c.astype(np.float64) <= exact)
    ulp = np.spacing(np.abs(exact).astype(np.float32)).astype(np.float64)
    assert np.all(exact - c.astype(np.float64) <= 2.0 * ulp)


def test_random_products(mul_down):
    rng = np.random.default_rng(1)
    for scale in (1.0, 1e3, 1e20):
        _check(mul_down, rng.uniform(-1, 1, 2_000_000) * 1e3, rng.uniform(-1, 1, 2_000_000) * scale + 1e-20)


def test_products_at_powers_of_two(mul_down):
    """Pairs whose rounded product is a power of two, of both signs, from above
    and from below."""
    rng = np.random.default_rng(2)
    a = rng.uniform(1, 2, 1_000_000).astype(np.float32)
    b = (1.0 / a.astype(np.float64)).astype(np.float32)
    for step in (-1, 0, 1):
        near = (b.view(np.int32) + step).view(np.float32)
        hit = np.abs(a * near) == 1.0
        assert hit.sum() > 1000 or step
        for sa in (1, -1):
            for p in (-30, 0, 17):
                _check(mul_down, sa * a[hit], np.ldexp(near[hit], p))
    _check(mul_down, np.float32([0.0, -0.0, 1.0, -1.0, 2.0]), np.float32([3.0, 3.0, 1.0, 1.0, -4.0]))
