"""How the block-by-block CBC decryption of message sets deals its messages to
waves (csrc/aes_cbc_flat_split.hpp, compiled here for the CPU): every message
to exactly one lane of one group, and no wave with more steps than one wave
per message, dealt in turn, would leave it, whatever the order of the
lengths."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1902_05234_amd import inputs

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1902_05234_amd", "csrc")
WRAPPER = """
#include "aes_cbc_flat_split.hpp"
static aesgpu::FlatSplit s;
extern "C" void split(uint64_t n, uint64_t in_blocks, int one_arena, int cus, uint64_t* out)
{
    s = aesgpu::flat_split(n, in_blocks, one_arena, cus);
    out[0] = s.groups, out[1] = s.per_group, out[2] = s.slices;
}
extern "C" void members(uint64_t* out)
{
    for (uint64_t g = 0; g < s.groups; ++g)
        for (uint32_t l = 0; l < s.per_group; ++l)
            *out++ = aesgpu::flat_message(s, g, l);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "w.cpp").write_text(WRAPPER)
    so = str(d / "w.so")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                        str(d / "w.cpp"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = ctypes.CDLL(so)
    lib.split.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    lib.members.argtypes = [ctypes.c_void_p]
    return lib


def split(lib, n, in_blocks, one_arena, cus):
    s = np.zeros(3, dtype=np.uint64)
    lib.split(n, in_blocks, one_arena, cus, s.ctypes.data)
    m = np.zeros(int(s[0] * s[1]), dtype=np.uint64)
    lib.members(m.ctypes.data)
    return [int(v) for v in s], m.astype(np.int64).reshape(int(s[0]), int(s[1]))


@pytest.mark.parametrize("cus", [1, 32, 256])
def test_every_message_in_one_group(lib, cus):
    g = inputs.rng(21, cus)
    sizes = [1, 2, 3, 63, 64, 65, 1000, 4095, 4096, 4097, 70000, 262144, 262145, 300001]
    for n in sizes + [int(x) for x in np.exp(g.uniform(0, np.log(3e5), 40))]:
        for mean in (0.3, 1, 5, 8, 31, 63, 64, 700):
            for one_arena in (0, 1):
                s, m = split(lib, n, int(n * mean), one_arena, cus)
                assert s[1] <= 64 and s[2] >= 1 and not (one_arena and s[2] > 1)
                assert s[2] == 1 or s[0] * s[2] <= 16 * cus
                seen = np.bincount(m.reshape(-1)[m.reshape(-1) < n], minlength=n)
                assert (seen == 1).all(), (n, mean, one_arena, s)
                assert (m[:, 1:] > m[:, :-1]).all()


def _waves(cost, resident):
    """Most steps of a wave when the units go to the resident waves in turn."""
    c = np.zeros(-(-cost.size // resident) * resident, dtype=np.int64)
    c[:cost.size] = cost
    return int(c.reshape(-1, resident).sum(0).max())


def _orders(n, hi):
    g = inputs.rng(22, n, hi)
    log = np.exp(g.uniform(0, np.log(hi), n)).astype(np.int64)
    heap = np.zeros(n, dtype=np.int64)
    heap[n // 3:n // 3 + 64] = 64 * n // 64 + hi
    yield "sorted", np.sort(log)
    yield "sorted down", np.sort(log)[::-1]
    yield "random", log
    yield "uniform sorted", np.sort(g.integers(0, hi + 1, n))
    yield "64 in a row", heap
    for period in (2, 3, 16, 64, 1024):
        yield "every %dth" % period, np.where(np.arange(n) % period == 1, hi, hi // 16)


@pytest.mark.parametrize("n,hi", [(4096, 4096), (5000, 4096), (8192, 1024), (16384, 65536), (65536, 600), (262144, 300)])
def test_no_wave_gets_more_than_one_wave_per_message_would(lib, n, hi):
    resident = 16 * 256
    for name, nb in _orders(n, hi):
        s, m = split(lib, n, int(nb.sum()), 0, 256)
        padded = np.append(nb, 0)
        steps = -(-padded[np.minimum(m, n)].sum(1) // 64)
        unit = np.maximum(0, -((np.arange(s[2])[None, :] - steps[:, None]) // s[2])).reshape(-1)
        assert unit.sum() == steps.sum()
        per_message = _waves(-(-nb // 64), resident)
        # one message longer than a wave's share sets the pace of both; a slice more is the rounding of a share
        assert _waves(unit, resident) <= per_message * 1.05 + 1, (name, s, per_message)
