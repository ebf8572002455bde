"""Geometry of the reconstruction in bands and the rule that chooses it, on the CPU: the header is plain C++."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = '''
#include "comet_bands.h"
using namespace comet;
extern "C" void geometry(uint64_t planes, uint32_t h, uint32_t w, uint32_t vec, uint64_t *out) {
    const BandGeom g = band_geometry(planes, h, w, vec);
    const uint64_t v[] = {g.R, g.segs, g.bands, g.n_units, g.off_row, g.off_unit, g.bytes};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
}
extern "C" uint64_t bytes_max(uint64_t n) { return band_bytes_max(n); }
extern "C" int pays(int num_cu, uint64_t planes, uint32_t h, uint32_t w, uint32_t vec, int chunk64) {
    return band_pays(num_cu, planes, h, w, band_geometry(planes, h, w, vec), chunk64 != 0);
}
'''


@pytest.fixture(scope="module")
def bands(tmp_path_factory):
    d = tmp_path_factory.mktemp("bands")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2111_09562_amd", "csrc"),
                           "-o", str(d / "shim.so"), str(d / "shim.cpp")])
    lib = C.CDLL(str(d / "shim.so"))
    lib.geometry.argtypes = [C.c_uint64, C.c_uint32, C.c_uint32, C.c_uint32, C.POINTER(C.c_uint64)]
    lib.bytes_max.argtypes, lib.bytes_max.restype = [C.c_uint64], C.c_uint64
    lib.pays.argtypes = [C.c_int, C.c_uint64, C.c_uint32, C.c_uint32, C.c_uint32, C.c_int]
    return lib


def _geometry(lib, planes, h, w, vec):
    out = (C.c_uint64 * 7)()
    lib.geometry(planes, h, w, vec, out)
    return [int(v) for v in out]


def _shapes():
    edge_h = [1, 2, 7, 8, 9, 15, 16, 17, 24, 31, 63, 64, 65, 127, 128, 129, 480, 1000, 65537, 2097151]
    edge_w = [128, 129, 130, 191, 192, 193, 255, 256, 257, 258, 511, 512, 513, 640, 854, 1025, 8191, 8192]
    for h in edge_h:
        for w in edge_w:
            for planes in (1, 3, 32, 4096, 100003):
                yield planes, h, w
    rng = random.Random(5)
    for _ in range(20000):
        w = int(128 * 64 ** rng.random())
        h = int(2 ** (21 * rng.random()))
        n = int(2 ** (31 * rng.random()))
        yield max(1, n // (w * h)), h, w


def test_bands_cover_the_plane_and_fit_the_workspace(bands):
    for planes, h, w in _shapes():
        n = planes * h * w
        if n > 2 ** 31 - 1:
            continue
        for vec in (1, 2) if w % 2 == 0 else (1,):
            R, segs, nb, units, off_row, off_unit, total = _geometry(bands, planes, h, w, vec)
            what = (planes, h, w, vec)
            assert 1 <= R <= 64 and (nb - 1) * R < h <= nb * R, what
            assert (segs - 1) * 64 * vec < w <= segs * 64 * vec and units == planes * nb * segs, what
            assert off_row >= 4 * planes * (nb - 1) * w and off_unit - off_row >= 4 * planes * nb * (segs - 1) * R, what
            assert total - off_unit >= (4 * units if nb > 1 and segs > 1 else 0), what
            assert total <= bands.bytes_max(n), what


def test_the_workspace_is_a_small_part_of_a_context(bands):
    """Every context holds it, also where no plane is wide: within a fourteenth of the two bytes per element that the
    codes take for large tensors, and a few megabytes for small ones."""
    for n in (1, 1000, 1 << 20, 1 << 22, 1 << 25):
        assert bands.bytes_max(n) <= min(n, 6 << 20) + 1024
    for n in (1 << 26, 411041792, 2 ** 31 - 1):
        assert bands.bytes_max(n) <= 2 * n / 14


# us with a plane per wavefront or workgroup / in bands, chunks of 64 symbols, two columns per lane where the width is even
MEASURED = [
    (4, 512, 512, 672, 48), (64, 512, 512, 721, 91), (1024, 512, 512, 848, 991),
    (256, 257, 257, 361, 99), (1024, 257, 257, 452, 340), (4096, 257, 257, 757, 1260),
    (8, 3000, 256, 265, 84), (512, 256, 256, 75, 127),
    # tall planes: a unit reads the column sums of all bands above it
    (60, 262143, 128, 11388, 19220), (60, 131071, 256, 11315, 12909), (15, 1048575, 128, 45452, 59022), (7, 2097151, 128, 90840, 132590),
    (3, 2097151, 128, 89885, 57094), (1, 2097151, 128, 87621, 19323), (7, 1048575, 256, 90228, 71856), (7, 524287, 512, 730577, 40801),
    (30, 262143, 128, 11296, 9732), (5, 2097151, 128, 90798, 93527), (1, 131072, 128, 5402, 352), (100, 8192, 512, 11461, 1476),
]


@pytest.mark.parametrize("planes,h,w,other,in_bands", MEASURED)
def test_the_rule_takes_the_quicker_way(bands, planes, h, w, other, in_bands):
    assert bool(bands.pays(256, planes, h, w, 2 - w % 2, 1)) == (in_bands < other)
