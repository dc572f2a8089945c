"""The error bound of the exact search's bf16 screening (csrc/exact_bound.h),
evaluated on the host: |dd - d| <= eps on rows whose bf16 roundings all point
one way, where it is nearly reached, and on random ones."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_22922_amd", "csrc")


@pytest.fixture(scope="module")
def eps(tmp_path_factory):
    d = tmp_path_factory.mktemp("exact_bound")
    src, lib = d / "b.cpp", d / "b.so"
    src.write_text('#include "exact_bound.h"\n'
                   'extern "C" float eps(int dim, double x, double xe, double q, double qe) {\n'
                   '  return ifvs::exact_eps(dim, x, xe, q, qe);\n}\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__host__=", "-D__device__=", "-I", CSRC, str(src),
                    "-o", str(lib)], check=True)
    fn = ctypes.CDLL(str(lib)).eps
    fn.argtypes, fn.restype = [ctypes.c_int] + [ctypes.c_double] * 4, ctypes.c_float
    return fn


def _bf16(a):
    u = a.astype(np.float32).view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(np.float32)


def _dd(x, q):
    """The screening's value for every row, its sums in fp32."""
    n2 = lambda a: np.add.accumulate(a * a, axis=-1, dtype=np.float32)[..., -1]
    dot = np.add.accumulate(_bf16(x) * _bf16(q), axis=-1, dtype=np.float32)[:, -1]
    return n2(x) + n2(q) - np.float32(2) * dot


def _rows(kind, dim, rng):
    up, down = 1 + 2.0 ** -8 + 2.0 ** -14, 1 + 2.0 ** -8       # rounded up and down by bf16
    if kind == "one way":
        q = np.full(dim, down)
        x = np.stack([np.full(dim, down), np.full(dim, up), np.where(np.arange(dim) < dim // 2, down, up)])
    elif kind == "scaled":
        q = down * 2.0 ** rng.integers(-8, 9, dim)
        x = q * 2.0 ** rng.integers(-1, 2, (200, 1)) * rng.choice([1.0, -1.0], (200, 1))
    else:
        q, x = rng.standard_normal(dim), rng.standard_normal((500, dim))
    return x.astype(np.float32), q.astype(np.float32)


@pytest.mark.parametrize("dim", [1, 16, 50, 96, 97, 128, 960])
@pytest.mark.parametrize("kind", ["one way", "scaled", "random"])
def test_bound_holds(eps, dim, kind):
    x, q = _rows(kind, dim, np.random.default_rng(dim))
    d = np.add.accumulate((x - q) ** 2, axis=-1, dtype=np.float32)[:, -1].astype(np.float64)
    norm = lambda a: np.sqrt((a.astype(np.float64) ** 2).sum(-1))
    moved = lambda a: norm(a.astype(np.float64) - _bf16(a).astype(np.float64))
    bound = eps(dim, norm(x).max(), moved(x).max(), norm(q), moved(q))
    err = np.abs(_dd(x, q).astype(np.float64) - d).max()
    assert err <= bound
    if kind == "one way" and dim >= 16:
        assert err > 0.9 * 2 * (2 ** -7) * norm(x).max() * norm(q) * (1 - 2 ** -8)   # nearly reached
