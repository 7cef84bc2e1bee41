"""The queue of donated tasks on the CPU: its slot arithmetic compiled for the host."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("donate") / "donate_host.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared",
                           os.path.join(HERE, "native", "donate_host.cpp"), "-o", out])
    L = ctypes.CDLL(out)
    for f in (L.t_slot, L.t_published, L.t_read, L.t_last):
        f.restype = ctypes.c_uint32
    for f in (L.t_slot, L.t_published, L.t_read):
        f.argtypes = [ctypes.c_uint32] * 2
    L.t_fits.argtypes = [ctypes.c_uint32] * 4
    return L


@pytest.mark.parametrize("cap", [4, 2048, 4096])
def test_ready_words_never_repeat_and_the_numbers_end(lib, cap):
    last = lib.t_last()
    for s in (0, 1, cap - 1, cap, 2 * cap + 3, last - cap, last):
        assert lib.t_slot(s, cap) == s % cap
        use = s // cap
        assert (lib.t_published(s, cap), lib.t_read(s, cap)) == (3 * use + 1, 3 * use + 3)
        if s + cap <= last:  # the next use starts where this one ended, and its words are larger
            assert lib.t_published(s + cap, cap) == lib.t_read(s, cap) + 1
    assert lib.t_fits(0, 0, min(64, cap), cap)
    assert lib.t_fits(5, 5 + cap - 3, 3, cap) and not lib.t_fits(5, 5 + cap - 3, 4, cap)
    assert lib.t_fits(last - 64, last - 64, min(64, cap), cap)
    assert not lib.t_fits(last, last, 1, cap) and not lib.t_fits(last - 2, last - 2, 3, cap)
