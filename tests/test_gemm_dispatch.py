"""Rules that pick a GEMM kernel and its split, as the library's host code
computes them (256 compute units where there is no device)."""
import ctypes as C
import functools
import os

import pytest

from paper_2609_01068_amd import build

F32, BF16, E4M3 = 0, 1, 2
STORE_F32, STORE_ACT, RESID, SWIGLU, PARTIAL, PARTIAL_TILE, QKV_ROPE = range(7)
WIDTHS = [n for n in range(512, 16385, 256)]


@functools.lru_cache(maxsize=None)
def library_host():
    if not os.path.exists(build.LIB_PATH):
        build.build(verbose=False)
    lib = C.CDLL(build.LIB_PATH)

    def function(name, params, result=C.c_int):
        f = getattr(lib, f"_ZN7outlets{len(name)}{name}E{params or 'v'}")
        f.restype = result
        f.argtypes = [{"i": C.c_int, "m": C.c_size_t}[p] for p in params]
        return f

    class Host:
        cus = function("gemm_device_cus", "")()
        streams = function("gemm_streams", "iiiii", C.c_bool)
        splits = function("gemm_splitk_plan", "iiiii")
        stream_workgroups = function("gemm_stream_workgroups", "iiii")
        workspace_bytes = function("gemm_workspace_bytes", "iiiiim", C.c_size_t)

    return Host


@pytest.fixture(scope="module")
def host():
    return library_host()


@pytest.mark.parametrize("fmt", [BF16, E4M3], ids=["bf16", "e4m3"])
def test_few_row_splits_fit_one_round(host, fmt):
    """A K split of the few-row kernel fills the CUs at most once."""
    for n in WIDTHS:
        for k in (n, 3 * n, 14336):
            for m in (1, 16, 33, 64):
                if not host.streams(fmt, RESID, m, n, k):
                    continue
                s = host.splits(fmt, RESID, m, n, k)
                if s > 1:
                    assert host.stream_workgroups(fmt, PARTIAL, n, s) <= host.cus, (n, k, m, s)


def test_few_row_bound_of_large_bf16_matrices(host):
    """From 33 rows, bf16 matrices past 64M weights go to the tiles."""
    for n, k, few in ((4096, 12288, True), (4096, 14336, True), (4096, 16384, True), (4096, 16640, False),
                      (5120, 15360, False), (6144, 18432, False)):
        assert host.streams(BF16, RESID, 32, n, k)
        assert host.streams(BF16, RESID, 33, n, k) == host.streams(BF16, RESID, 64, n, k) == few, (n, k)
        assert host.streams(E4M3, RESID, 64, n, k)
