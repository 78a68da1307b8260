"""Host arithmetic of the TOA pass (no GPU): the chunks of ragged data sets, the
waves that share one, and how far the kernel's loads reach past the last TOA, by
the kernel's own walk over a chunk (a wave loads its first tile, and during each
tile the next one, before it looks whether there is one)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_06834_amd", "csrc")

SOURCE = """
#include "toa_chunks.h"
extern "C" int pad() { return pt::kToaPad; }
extern "C" int chunks(const int64_t *off, int n, int tpc, int32_t *begin, int32_t *end, int *max_tiles) {
  const pt::ToaChunks c = pt::cut_chunks(off, n, tpc);
  std::copy(c.begin.begin(), c.begin.end(), begin);
  std::copy(c.end.begin(), c.end.end(), end);
  *max_tiles = c.max_tiles;
  return (int)c.psr.size();
}
extern "C" int waves(int tuned, int waves, int max_tiles, int n_chunks, int n_cu) {
  return pt::toa_waves(tuned, waves, max_tiles, n_chunks, n_cu);
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("toa_chunks")
    (d / "host.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "host.cpp"), "-o",
                    str(d / "host.so")], check=True)
    return ctypes.CDLL(str(d / "host.so"))


def cut(host, counts, tpc):
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    room = int(np.sum(counts)) // 16 + 2 * len(counts)
    b, e, mt = np.zeros(room, np.int32), np.zeros(room, np.int32), ctypes.c_int()
    n = host.chunks(off.ctypes.data_as(ctypes.c_void_p), len(counts), tpc, b.ctypes.data_as(ctypes.c_void_p),
                    e.ctypes.data_as(ctypes.c_void_p), ctypes.byref(mt))
    return b[:n], e[:n], mt.value


def last_read(tb, te, waves):
    """Largest index that the waves of the chunk [tb, te) load."""
    top = 0
    for w in range(waves):
        base = tb + 16 * w
        top = max(top, base + 15)
        while base < te:
            top = max(top, base + 16 * waves + 15)
            base += 16 * waves
    return top


COUNTS = [[500] * 3, [497] * 3, [150], [1], [16], [17], [40, 1], [1500, 1], [2048, 1000, 241]] + \
    [[300, 16 * tiles + r] for tiles in (0, 1, 7, 8, 16, 31) for r in range(1, 17)]


@pytest.mark.parametrize("tuned", [0, 1, 2, 4, 8])   # (0: the rule)
@pytest.mark.parametrize("tpc", [1, 4, 9, 16, 33, 96, 4096])
def test_loads_stay_in_the_arrays(host, tpc, tuned):
    for counts in COUNTS:
        b, e, mt = cut(host, counts, tpc)
        assert b[0] == 0 and e[-1] == sum(counts) and np.all(e > b) and np.all(b[1:] == e[:-1])
        assert mt == np.max((e - b + 15) // 16) <= tpc
        for n_cu in (1, 64, 256, 1 << 20):
            w = host.waves(tuned > 0, tuned or 1, mt, len(b), n_cu)
            top = max(last_read(int(tb), int(te), w) for tb, te in zip(b, e))
            assert top < sum(counts) + host.pad(), (counts, tpc, tuned, n_cu, w)


def test_waves_rule(host):
    """A caller's number of waves is taken as it is; the rule never gives a wave
    less than a tile of the longest chunk, nor more than one wave to many chunks."""
    n_cu = 256
    for n in range(1, 300):
        for tiles in range(1, 40):
            for w in (1, 2, 4):
                assert host.waves(1, w, tiles, n, n_cu) == w
            w = host.waves(0, 1, tiles, n, n_cu)
            assert w in (1, 2, 4, 8) and w <= tiles and (w == 1 or 3 * n < n_cu)
    assert [host.waves(0, 1, 16, n, n_cu) for n in (6, 31, 32, 85, 86, 150)] == [8, 8, 4, 4, 1, 1]
    assert [host.waves(0, 1, 8, n, n_cu) for n in (31, 32, 86)] == [8, 4, 1]
    assert [host.waves(0, 1, 7, n, n_cu) for n in (16, 17)] == [2, 1] and host.waves(0, 1, 3, 2, n_cu) == 1
