"""The GELU forms of the device header on the CPU: their text is compiled with the
host's exp2 and division in place of the hardware's exp2 and reciprocal (all
within one unit in the last place) and compared with float64 and with the tanhf
forms of the same header."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_16074_amd", "csrc",
                      "jn_device.h")


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    text = open(HEADER).read()
    text = text[text.index("// tanh-form GELU and its derivative"): text.index("}  // namespace jnx")]
    names = [n for n in ("gelu_f", "gelu_exact_f", "gelu_grad_f", "gelu_grad_fast_f") if f" {n}(float u)" in text]
    src = ("#include <cmath>\n#define __device__\n#define __forceinline__ inline\n"
           "static float __builtin_amdgcn_exp2f(float x) { return x < -126.f ? 0.f : exp2f(x); }\n"
           "static float __builtin_amdgcn_rcpf(float x) { return 1.f / x; }\n" + text)
    for n in names:
        src += (f'extern "C" void run_{n}(const float* x, float* y, long n) '
                f"{{ for (long i = 0; i < n; ++i) y[i] = {n}(x[i]); }}\n")
    tmp = tmp_path_factory.mktemp("gelu")
    (tmp / "f.cpp").write_text(src)
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=fast", "-shared", "-fPIC", str(tmp / "f.cpp"), "-o",
                    str(tmp / "f.so")], check=True)
    so = ctypes.CDLL(str(tmp / "f.so"))

    def call(name, x):
        x = np.ascontiguousarray(x, dtype=np.float32)
        y = np.empty_like(x)
        getattr(so, "run_" + name)(x.ctypes.data_as(ctypes.c_void_p), y.ctypes.data_as(ctypes.c_void_p),
                                   ctypes.c_long(x.size))
        return y
    return call


def exact(u):
    c = np.sqrt(2 / np.pi)
    t = np.tanh(c * (u + 0.044715 * u ** 3))
    return 0.5 * u * (1 + t), 0.5 * (1 + t) + 0.5 * u * (1 - t * t) * c * (1 + 3 * 0.044715 * u * u)


def test_derivative_of_large_values(forms):
    """Where the tanhf form has saturated: 1 above, nothing below, no overflow; NaN stays NaN."""
    big = np.array([12, 20, 1e3, 1e6, 1e12, 1e13, 1e14, 1e18, 1e30, 3e38, np.inf], dtype=np.float32)
    assert np.array_equal(forms("gelu_grad_fast_f", big), np.ones_like(big))
    assert np.max(np.abs(forms("gelu_grad_fast_f", -big))) < 1e-34
    assert np.isnan(forms("gelu_grad_fast_f", [np.nan]))
    tame = big[big < 1e18]
    assert np.max(np.abs(forms("gelu_grad_fast_f", -tame) - forms("gelu_grad_f", -tame))) < 1e-34


@pytest.mark.parametrize("sigma", [0.5, 0.64, 1.0, 3.0])
def test_derivative_is_no_less_exact_than_the_tanhf_form(forms, sigma):
    u = np.random.default_rng(1).normal(0, sigma, 1 << 20).astype(np.float32)
    ref = exact(u.astype(np.float64))[1]
    fast, form = (np.linalg.norm(forms(n, u) - ref) for n in ("gelu_grad_fast_f", "gelu_grad_f"))
    assert fast <= form, (fast / np.linalg.norm(ref), form / np.linalg.norm(ref))


def test_value_of_large_values(forms):
    big = np.array([12, 20, 1e3, 1e6, 1e13, 1e30, 3e38, np.inf], dtype=np.float32)
    assert np.array_equal(forms("gelu_exact_f", big), big)
    assert np.array_equal(np.isnan(forms("gelu_exact_f", -big)), np.isinf(big))  # as the tanhf form
    assert np.max(np.abs(forms("gelu_exact_f", -big[:-1]))) < 1e-34
    assert np.isnan(forms("gelu_exact_f", [np.nan]))


@pytest.mark.parametrize("sigma", [0.3, 0.5, 0.64, 1.0, 3.0])
def test_value_is_no_less_exact_than_the_tanhf_form(forms, sigma):
    u = np.random.default_rng(1).normal(0, sigma, 1 << 20).astype(np.float32)
    ref = exact(u.astype(np.float64))[0]
    fast, form = (np.linalg.norm(forms(n, u) - ref) for n in ("gelu_exact_f", "gelu_f"))
    assert fast <= form, (fast / np.linalg.norm(ref), form / np.linalg.norm(ref))


def test_the_saved_gelu_takes_that_form():
    gemm = open(os.path.join(os.path.dirname(HEADER), "k_gemm.hip")).read()
    at = gemm.index("EPI == EPI_GELU_SAVE) {")
    assert "gelu_exact_f(" in gemm[at: at + 400]
