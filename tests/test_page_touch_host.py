"""Mapping a read-out array's pages before the copies (no GPU;
csrc/host_common.hpp compiled for the host alone): a fresh array's pages are all
mapped, a kept array's are left alone, values stay."""
import ctypes
import mmap
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "host_common.hpp"
// a fresh mapping whose first `kept` bytes are in memory: the bytes that
// touch_pages went over, and what a second call went over
extern "C" void touched(size_t bytes, size_t kept, long *first, long *second, long *resident)
{
    char *p = (char *)mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    madvise(p, bytes, MADV_NOHUGEPAGE);
    for (size_t i = 0; i < kept; i += 4096) p[i] = 1;
    *first = (long)lbm::touch_pages((double *)p, bytes);
    *second = (long)lbm::touch_pages((double *)p, bytes);
    std::vector<unsigned char> in((bytes + 4095) / 4096);
    *resident = mincore(p, bytes, in.data()) ? -1 : 0;
    for (unsigned char c : in) *resident += c & 1;
    munmap(p, bytes);
}
extern "C" long piece() { return (long)lbm::kTouchPiece; }
extern "C" long touch(void *a, size_t bytes) { return (long)lbm::touch_pages((double *)a, bytes); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    assert mmap.PAGESIZE == 4096
    d = tmp_path_factory.mktemp("touch")
    src, so = d / "touch.cpp", d / "touch.so"
    src.write_text(SOURCE)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "paper_2208_13769_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lp = ctypes.POINTER(ctypes.c_long)
    lib.piece.restype = lib.touch.restype = ctypes.c_long
    lib.touched.argtypes = [ctypes.c_size_t, ctypes.c_size_t, lp, lp, lp]
    lib.touch.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    return lib


def _touched(lib, bytes_, kept):
    out = [ctypes.c_long() for _ in range(3)]
    lib.touched(bytes_, kept, *(ctypes.byref(o) for o in out))
    return tuple(o.value for o in out)


def test_fresh_pages_are_mapped_once(lib):
    for bytes_ in (8, 4096, 4104, 2 * lib.piece(), 5 * lib.piece() + 3 * 4096 + 24):
        assert _touched(lib, bytes_, 0) == (bytes_, 0, -(-bytes_ // 4096))


def test_kept_pages_are_left_alone(lib):
    n = 4 * lib.piece() + 4096
    assert _touched(lib, n, n) == (0, 0, n // 4096)
    assert _touched(lib, n, 2 * lib.piece())[:2] == (n - 2 * lib.piece(), 0)


def test_values_stay(lib):
    want = np.arange(700001, dtype=np.float64)
    a = want.copy()
    assert lib.touch(a.ctypes.data, a.nbytes) == 0
    assert np.array_equal(a, want)
    b = np.zeros(700001)
    assert lib.touch(b.ctypes.data, b.nbytes) >= 0
    assert not b.any()
