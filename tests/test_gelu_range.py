"""The fp32 GELU and its derivative as the kernels have them (compiled for the host), over the whole range of fp32 arguments, against
64 bits.  Beyond |z| = 14 the derivative is 0 or 1 to the last bit: a diverging replica, or a bias used as a switch, must not turn it into
something that grows with z."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def gelu(tmp_path_factory):
    text = open(os.path.join(ROOT, "paper_2604_24708_amd", "csrc", "hdet_elem.h")).read()
    names = ("hdet_gelu_exp", "hdet_gelu_sigma_fast", "hdet_gelu_tanh", "hdet_gelu_tanh_grad", "hdet_gelu_tanh_fast", "hdet_gelu_tanh_grad_fast")
    bodies = [re.search(r"__device__ __forceinline__ float %s\(.*?\n}\n" % n, text, re.S).group(0) for n in names]
    loops = "".join('extern "C" void %s_all(const float* x, float* y, long n) { for (long i = 0; i < n; ++i) y[i] = %s(x[i]); }\n' % (n, n)
                    for n in names[2:])
    d = tmp_path_factory.mktemp("gelu")
    src = d / "gelu.cpp"
    builtins = ("static float __builtin_amdgcn_rcpf(float x) { return 1.f / x; }\n"
                "static float __builtin_amdgcn_exp2f(float x) { return exp2f(x); }\n"
                "static float __builtin_amdgcn_fmed3f(float x, float a, float b) { return fmaxf(fminf(fmaxf(x, a), b), a); }\n")
    src.write_text("#include <cmath>\n#define __device__\n#define __forceinline__ inline\n" + builtins + "".join(bodies) + loops)
    cc = shutil.which("g++")
    assert cc, "g++ not found"
    lib = str(d / "gelu.so")
    subprocess.run([cc, "-O1", "-ffp-contract=off", "-shared", "-fPIC", str(src), "-o", lib], check=True)
    dll = ctypes.CDLL(lib)

    def call(name, x):
        x = np.ascontiguousarray(x, np.float32)
        y = np.empty_like(x)
        f = getattr(dll, name + "_all")
        f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long]
        f(x.ctypes.data, y.ctypes.data, x.size)
        return y

    return call


def exact(z):
    z = np.asarray(z, np.float64)
    c = np.sqrt(2.0 / np.pi)
    with np.errstate(over="ignore", invalid="ignore"):
        e = np.exp(np.minimum(-2.0 * c * (z + 0.044715 * z ** 3), 700.0))
        s = 1.0 / (1.0 + e)
        value = np.where(z < -14, 0.0, z * s)
        grad = np.where(z < -14, 0.0, np.where(z > 14, 1.0, s * (1.0 + z * (e * s) * 2.0 * c * (1.0 + 3 * 0.044715 * z * z))))
    return value, grad


def everywhere():
    size = np.concatenate([np.logspace(-38, np.log10(3.4e38), 4001), np.linspace(0.01, 14, 4001), [9.99, 10.0, 10.01, np.inf]]).astype(np.float32)
    return np.concatenate([-size, size])


def test_range_of_the_fast_derivative(gelu):
    z = everywhere()
    got, grad = gelu("hdet_gelu_tanh_grad_fast", z), exact(z)[1]
    # 1 - sigma of a rounded sigma, times z 2 u' (up to 30 where it counts): rounded to bfloat16 afterwards
    assert np.all(np.isfinite(got)) and np.max(np.abs(got - grad)) <= 5e-6, z[np.argmax(np.abs(got - grad))]


def test_range(gelu):
    z = everywhere()
    value, grad = exact(z)
    got = gelu("hdet_gelu_tanh_grad", z)
    # the derivative is between -0.13 and 1.13: a few roundings of numbers of that size
    assert np.all(np.isfinite(got)) and np.max(np.abs(got - grad)) <= 5e-7, z[np.argmax(np.abs(got - grad))]
    assert np.all(got[z < -14] == 0) and np.all(got[z > 14] == 1)
    ok = np.isfinite(z)
    got = gelu("hdet_gelu_tanh", z)[ok]
    # exp(-2u) carries the rounding of 2u, which is at most 14 where the value matters
    assert np.all(np.isfinite(got)) and np.max(np.abs(got - value[ok]) / (np.abs(value[ok]) + 1e-5)) <= 5e-6


@pytest.mark.parametrize("size,value_bound,grad_bound", [(1.0, 2.1e-8, 5e-8), (2.0, 3.9e-8, 5e-8)])
def test_ordinary_arguments(gelu, size, value_bound, grad_bound):
    """rms over normal arguments: little more than the result's own rounding (1.7e-8 and 3.4e-8) for the value, a few roundings of numbers up to 1
    for the derivative."""
    z = (size * np.random.Generator(np.random.Philox(5)).standard_normal(200000)).astype(np.float32)
    value, grad = exact(z)
    assert np.sqrt(np.mean((gelu("hdet_gelu_tanh", z) - value) ** 2)) <= value_bound
    assert np.sqrt(np.mean((gelu("hdet_gelu_tanh_grad", z) - grad) ** 2)) <= grad_bound


def test_infinity(gelu):
    assert gelu("hdet_gelu_tanh", np.array([np.inf], np.float32))[0] == np.inf


def test_nan_stays(gelu):
    z = np.array([np.nan, -np.nan], np.float32)
    assert np.all(np.isnan(gelu("hdet_gelu_tanh", z))) and np.all(np.isnan(gelu("hdet_gelu_tanh_grad", z)))
