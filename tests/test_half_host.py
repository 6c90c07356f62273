"""The host's half-precision conversions equal numpy's, bit for bit."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2402_09633_amd import build as B


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("half")
    src, so = d / "half.cpp", d / "half.so"
    src.write_text('#include "half_host.h"\nextern "C" {\n'
                   "void to_half(const float *x, uint16_t *y, long n) { gnn::to_f16(x, y, n); }\n"
                   "void to_float(const uint16_t *x, float *y, long n) { gnn::to_f32(x, y, n); }\n"
                   "void split(const double *x, uint16_t *y, long n) {\n"
                   "  for (; n > 0; n -= 64, x += 64, y += 192)\n"
                   "    gnn::split_f16<3>(*(const double(*)[64])x, y);\n}\n}\n")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(B.CSRC), str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def convert(fn, x, dtype):
    y = np.empty(x.size, dtype)
    fn(x.ctypes.data_as(ctypes.c_void_p), y.ctypes.data_as(ctypes.c_void_p), ctypes.c_long(x.size))
    return y


def test_every_half_and_what_rounds_to_it(lib):
    h = np.arange(1 << 16, dtype=np.uint16)
    f = h.view(np.float16).astype(np.float32)
    ok = ~np.isnan(f)
    got = convert(lib.to_float, h, np.float32)
    assert np.array_equal(got.view(np.uint32)[ok], f.view(np.uint32)[ok])
    assert np.isnan(got[~ok]).all()
    # around every half and every middle between two: +-2 in the last place
    # of fp32, and random bits
    fin = f[np.isfinite(f)]
    mid = ((np.sort(fin)[1:].astype(np.float64) + np.sort(fin)[:-1]) / 2).astype(np.float32)
    base = np.concatenate([fin, mid, np.float32([65504, 65519.996, 65520, 65536, 1e30])])
    u = base.view(np.uint32).astype(np.int64)
    bits = np.concatenate([u + k for k in range(-2, 3)] +
                          [np.random.default_rng(0).integers(0, 1 << 32, 1 << 20)])
    x = (bits % (1 << 32)).astype(np.uint32).view(np.float32)
    with np.errstate(over="ignore", invalid="ignore"):
        want = x.astype(np.float16)
    got = convert(lib.to_half, np.ascontiguousarray(x), np.uint16).view(np.float16)
    nan = np.isnan(x)
    assert np.array_equal(got.view(np.uint16)[~nan], want.view(np.uint16)[~nan])
    assert np.isnan(got[nan]).all()


def test_split_parts(lib):
    # (with the CPU's conversion where it has one)
    rng = np.random.default_rng(1)
    w = rng.normal(size=64 * 50) * 2.0 ** rng.integers(-30, 14, 64 * 50)
    got = np.empty(w.size * 3, np.uint16)
    lib.split(w.ctypes.data_as(ctypes.c_void_p), got.ctypes.data_as(ctypes.c_void_p),
              ctypes.c_long(w.size))
    left = w.reshape(-1, 64).copy()
    for p in range(3):
        want = left.astype(np.float32).astype(np.float16)
        part = got.reshape(-1, 3, 64)[:, p].view(np.float16)
        assert np.array_equal(part.view(np.uint16), want.view(np.uint16))
        left -= want.astype(np.float64)


def test_build_asks_for_no_host_cpu_feature():
    """The library loads on any host of its architecture."""
    assert not [f for f in B.FLAGS if f.startswith("-m")]
