"""The selection of the separate kernels (prr_topk.h), compiled for the CPU with its workgroup as
256 fibers (tests/host/prr_device.h): results against a sort, and that it ends whatever it reads."""
from __future__ import annotations

import ctypes
import os
import shutil
import subprocess
import zlib

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(HERE, "..", "paper_2606_30389_amd", "csrc", "prr_topk.h")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("topk_host")
    for src in (HEADER, os.path.join(HERE, "host", "prr_device.h"), os.path.join(HERE, "host", "topk_host.cpp")):
        shutil.copy(src, d)
    (d / "prr_launch.h").write_text("#pragma once\n#define PRR_MAX_PAGES_DEV 16384\n")
    lib = d / "topk_host.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", str(lib), str(d / "topk_host.cpp")], check=True)
    return ctypes.CDLL(str(lib))


def keys_of(x):
    u = (np.asarray(x, dtype=np.float32) + np.float32(0)).view(np.uint32)
    return np.where(u & 0x80000000, ~u, u | np.uint32(0x80000000)).astype(np.uint32)


def select(host, keys, k, forced=(), gmax=None, fill=0):
    """(ends, selected pages) of topk_select with a budget of k pages beside the forced ones."""
    n, shift = len(keys), host.topk_shift(len(keys))
    if gmax is None:
        pad = np.zeros(-n % (1 << shift), dtype=np.uint32)
        gmax = np.concatenate([keys, pad]).reshape(-1, 1 << shift).max(axis=1)
    f, out, count = np.asarray(forced, dtype=np.int32), np.full(1024, -7, dtype=np.int32), np.zeros(1, dtype=np.int32)
    keys, gmax = np.ascontiguousarray(keys), np.ascontiguousarray(gmax)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    rc = host.topk_host(n, shift, k, p(f), len(f), p(keys), p(gmax), p(out), 1024, p(count), fill)
    return rc == 0, out[:count[0]]


def values(dist, n, rng):
    x = rng.standard_normal(n)
    if dist == "constant":
        x[:] = 3.0
    elif dist == "levels":
        x = np.floor(6 * rng.random(n))
    elif dist == "near":
        x = 45.0 + 1e-5 * x
    elif dist == "cluster":
        x[n // 3:n // 3 + n // 4] += 8
    elif dist == "special":
        x[::7], x[1::7], x[2::7], x[3::7] = np.inf, -np.inf, np.nan, -0.0
    elif dist == "wide":
        x = np.sign(x) * 10.0 ** (30 * rng.random(n))
    return x.astype(np.float32)


@pytest.mark.parametrize("dist", ["gauss", "constant", "levels", "near", "cluster", "special", "wide"])
@pytest.mark.parametrize("n,k", [(5, 3), (700, 60), (2048, 1000), (2049, 1), (4100, 250), (8200, 512), (16384, 1000)])
def test_topk_select(host, dist, n, k):
    rng = np.random.default_rng(zlib.crc32(f"{dist}{n}".encode()))
    keys = keys_of(values(dist, n, rng))
    for forced in ([], sorted({0, n // 2, n - 1})):
        order = [p for p in np.argsort(-keys.astype(np.int64), kind="stable") if p not in forced]
        want = np.sort(np.concatenate([order[:k], forced]).astype(np.int64))
        ends, got = select(host, keys, k, forced, fill=0xA5)
        assert ends and np.array_equal(got, want)


@pytest.mark.parametrize("n,k", [(2500, 100), (8192, 256), (16384, 900)])
def test_topk_select_ends_on_groups_that_are_not_its_keys(host, n, k):
    """Group maxima that promise more pages than there are (a workspace that is written while
    it is in use, or was never zeroed): the list is then not the selection, but it is made."""
    rng = np.random.default_rng(n)
    ng = (n + (1 << host.topk_shift(n)) - 1) >> host.topk_shift(n)
    x = keys_of(rng.standard_normal(n))
    for keys, gmax in ((x, keys_of(100 + rng.standard_normal(ng))), (np.zeros(n, np.uint32), keys_of(rng.standard_normal(ng))),
                       (x, np.full(ng, 0xffffffff, np.uint32)), (x, np.zeros(ng, np.uint32)),
                       (x, rng.integers(0, 1 << 32, ng, dtype=np.uint32))):
        for fill in (0, 0xA5, 0x7F, 0xFF):
            ends, got = select(host, keys, k, gmax=gmax, fill=fill)
            assert ends, "the selection does not end"
            assert len(got) <= 1024 and np.all((got == -7) | ((got >= 0) & (got < n)))
