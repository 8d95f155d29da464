"""The directly evaluated factors of GeLU and its derivative, compiled for the host, against 64 bits: over every bf16 value and a grid of
32-bit ones, with the infinities and NaN, and no further off than the tables of the persistent kernels."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
from scipy.special import erfc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "gauss.h"
extern "C" void cdf(const float* z, float* out, long n) { for (long i = 0; i < n; ++i) out[i] = moe::normal_cdf(z[i]); }
extern "C" void slope(const float* z, float* out, long n) { for (long i = 0; i < n; ++i) out[i] = moe::gelu_slope(z[i]); }
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    where = tmp_path_factory.mktemp("gauss")
    (where / "gauss.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++20", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2103_13262_amd", "csrc"),
                    str(where / "gauss.cpp"), "-o", str(where / "gauss.so")], check=True)
    lib = ctypes.CDLL(str(where / "gauss.so"))

    def call(name, z):
        z, out = np.ascontiguousarray(z, np.float32), np.empty(len(z), np.float32)
        at = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        getattr(lib, name)(at(z), at(out), ctypes.c_long(len(z)))
        return out
    return call


def phi(z):
    return np.exp(-0.5 * z * z) / np.sqrt(2 * np.pi)


def Phi(z):
    return 0.5 * erfc(-z / np.sqrt(2))


def to_bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return (((u + 0x7fff + ((u >> 16) & 1)) >> 16 << 16).astype(np.uint32)).view(np.float32)


BF16 = (np.arange(65536, dtype=np.uint32) << 16).view(np.float32)
BF16 = BF16[np.isfinite(BF16)]


def test_cdf(host):
    z = np.concatenate([np.linspace(-9, 9, 400001), BF16]).astype(np.float32)
    z64 = z.astype(np.float64)
    err = host("cdf", z).astype(np.float64) - Phi(z64)
    # half of the last of 24 bits three times over (the complement, the power, their product) of a value up to 1
    assert abs(err).max() < 1.3e-7
    # below zero the power's argument, up to 41, is rounded to 24 bits: 2^-24 * 41 * ln 2 * 2 and the complement's cancellation from 1/2
    low = (z >= -9) & (z < 0)
    assert abs(err[low] / Phi(z64[low])).max() < 1e-5


def test_slope(host):
    z64 = BF16.astype(np.float64)
    err = host("slope", BF16).astype(np.float64) - (Phi(z64) + np.where(abs(z64) < 40, z64 * phi(np.clip(z64, -40, 40)), 0))
    assert abs(err).max() < 1.3e-7


def test_infinities_and_nan(host):
    z = np.array([np.inf, -np.inf, np.nan, 3e38, -3e38, 0.0, -0.0], np.float32)
    for name in ("cdf", "slope"):
        assert np.array_equal(host(name, z), np.array([1, 0, np.nan, 1, 0, 0.5, 0.5], np.float32), equal_nan=True), name


def test_no_further_off_than_the_tables(host):
    """H after its rounding to bf16, by interval of z, and the derivative's factor over pre-activations N(0, 0.64)."""
    rng = np.random.default_rng(0)
    table = lambda f, z: f(np.clip(np.abs(z), 2.0 ** -11, 8 * (1 - 2.0 ** -8)) * np.where(z < 0, -1.0, 1.0))
    for lo in range(-8, 8):
        z = rng.uniform(lo, lo + 1, 200000).astype(np.float32)
        z64, zb = z.astype(np.float64), to_bf16(z).astype(np.float64)
        ref = z64 * Phi(z64)
        rel = lambda h: np.sqrt(np.mean((to_bf16(h).astype(np.float64) / ref - 1) ** 2))
        looked_up = z64 * (table(Phi, zb) + (z64 - zb) * phi(zb))
        assert rel(z * host("cdf", z)) <= 1.01 * rel(looked_up), lo
    z = to_bf16(rng.normal(0, 0.64, 400000))
    z64 = z.astype(np.float64)
    ref = Phi(z64) + z64 * phi(z64)
    rms = lambda s: np.sqrt(np.mean((s - ref) ** 2))
    assert rms(host("slope", z)) <= rms(table(lambda v: Phi(v) + v * phi(v), z64).astype(np.float32))
