"""The refinements of the hardware's reciprocal and square-root estimates (csrc/refine.h), on the
host: within 0.5 ulp and a hundredth of the exact value from any estimate within 2^-24.

Derivation: the last step of each adds a correction of relative size 2^-47 or less, so its own
error is far below an ulp and the final rounding's half ulp remains (a hundredth allowed)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_36383_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("refine")
    src, so = d / "r.cpp", d / "r.so"
    src.write_text('#include "refine.h"\n'
                   'extern "C" void rcp(const double* x, const double* e, double* o, long n) {\n'
                   "  for (long i = 0; i < n; ++i) o[i] = gmhc::refined_rcp(x[i], e[i]);\n}\n"
                   'extern "C" void sqr(const double* x, const double* e, double* o, long n) {\n'
                   "  for (long i = 0; i < n; ++i) o[i] = gmhc::refined_sqrt(x[i], e[i]);\n}\n")
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-D__host__=", "-D__device__=",
                    "-D__forceinline__=inline", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return C.CDLL(str(so))


@pytest.mark.parametrize("op", ["rcp", "sqr"])
@pytest.mark.parametrize("err", [-1.0, -0.3, 0.0, 0.3, 1.0])
def test_refined_to_half_an_ulp(lib, op, err):
    rng = np.random.default_rng(11)
    n = 200000
    x = rng.uniform(1.0, 4.0, n) * 2.0 ** (2 * rng.integers(-40, 40, n))
    xl = x.astype(np.longdouble)
    exact = 1 / xl if op == "rcp" else np.sqrt(xl)
    est = (1 / xl if op == "rcp" else 1 / np.sqrt(xl)) * (1 + np.longdouble(err) * np.longdouble(2.0) ** -24)
    est = est.astype(np.float64)
    out = np.empty(n)
    ptr = [a.ctypes.data_as(C.c_void_p) for a in (x, est, out)]
    getattr(lib, op)(*ptr, C.c_long(n))
    ulp = np.spacing(exact.astype(np.float64)).astype(np.longdouble)
    worst = float(np.max(np.abs(out.astype(np.longdouble) - exact) / ulp))
    print(f"{op} from estimates off by {err} 2^-24: {worst:.4f} ulp")
    assert worst <= 0.51
