"""The run's host-side decisions (csrc/kp_rules.hpp), compiled on their own."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_01283_amd", "csrc")


def compiled(tmp, source):
    src, lib = os.path.join(tmp, "rules.cpp"), os.path.join(tmp, "librules.so")
    with open(src, "w") as f:
        f.write('#include "kp_rules.hpp"\n' + source)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib],
                   check=True)
    return C.CDLL(lib)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    z = C.c_size_t
    dll = compiled(str(tmp_path_factory.mktemp("rules")), """
using namespace kp;
extern "C" {
int copies(int c, size_t tally, size_t per, size_t have, size_t other, size_t free_b) {
  return copies_that_fit(c, tally, per, have, other, free_b);
}
int events(int batch, int lanes, int nactive, int exhausted, int peel) {
  return events_together(batch, lanes, nactive, exhausted, peel);
}
void pixels(unsigned npx, unsigned npy, int* xy) {
  for (unsigned p = 0; p < npx * npy; ++p) image_pixel(p, npx, npy, xy[2 * p], xy[2 * p + 1]);
}
int lanes(size_t total, size_t blocks, int waves) { return packets_per_wave(total, blocks, waves); }
size_t waves(size_t npix, size_t maps) { return (size_t)image_waves(npix, maps); }
size_t grow(size_t need, size_t have, size_t elem) { return grow_bytes(need, have, elem); }
}
""")
    dll.copies.argtypes = [C.c_int, z, z, z, z, z]
    dll.lanes.argtypes = [z, z, C.c_int]
    dll.waves.argtypes, dll.waves.restype = [z, z], z
    dll.grow.argtypes, dll.grow.restype = [z, z, z], z
    return dll


def test_a_held_tally_is_not_refused_for_its_copies(lib):
    """A context that holds the tally of a run below the copies' threshold, with
    less free memory than another tally: nothing has to be allocated."""
    assert lib.copies(8, 1000, 10, 1000, 0, 7999) == 0
    assert lib.copies(8, 1000, 10, 1000, 0, 8 * 1080 - 1) == 0
    assert lib.copies(8, 1000, 10, 1000, 0, 8 * 1080) == 8
    assert lib.copies(8, 1000, 10, 1080, 0, 0) == 8  # room is left in the buffer
    assert lib.copies(0, 1000, 10, 1000, 0, 0) == 0


def test_copies_never_refuse_a_run(lib):
    """Whatever is held and free, a run that fits without copies fits with those it gets."""
    n = 0
    for tally in (0, 5, 64, 100):
        for have in (0, 4, 64, 100, 120, 400):
            for other in (0, 8, 200):
                for free in range(0, 2200, 13):
                    for want in (0, 2, 32):
                        if lib.grow(tally, have, 8) + other > free:
                            continue
                        got = lib.copies(want, tally, 7, have, other, free)
                        assert got in (0, want)
                        assert lib.grow(tally + 7 * got, have, 8) + other <= free
                        n += got > 0
    assert n > 1000


def test_the_copied_box_without_overflow(tmp_path):
    """Every cell against boxes inside, across and outside the grid, and against
    none, in constant expressions: the compiler refuses one that overflows."""
    compiled(str(tmp_path), """
#include <initializer_list>
using namespace kp;
constexpr bool in(int cell, int low) { return hot_index(cell, low) < (uint32_t)HOT_SIDE; }
constexpr bool all(int n) {
  for (int c = 0; c < n; ++c) {
    if (in(c, HOT_NONE)) return false;
    for (int low : {-HOT_SIDE, -HOT_SIDE + 1, -1, 0, 1, 17, n - 1, n})
      if (in(c, low) != (c >= low && c < low + HOT_SIDE)) return false;
  }
  return true;
}
static_assert(all(40));
static_assert(!in(2147483647, HOT_NONE) && in(2147483647, 2147483640));
""")


def test_scattering_events_together(lib):
    """The setting's share of the lanes in use, or of the packets left; with
    peel-off, whose events cost far more than the steps meanwhile, the setting."""
    for batch in (1, 8, 64):
        assert lib.events(batch, 64, 64, 0, 0) == batch
        for lanes in (1, 29, 64):
            for nactive in range(1, lanes + 1):
                assert lib.events(batch, lanes, nactive, 0, 0) == batch * lanes // 64
                assert lib.events(batch, lanes, nactive, 1, 0) == batch * nactive // 64
                assert lib.events(batch, lanes, nactive, 0, 1) == lib.events(batch, lanes, nactive, 1, 1) == batch


def pixels(lib, npx, npy):
    xy = np.full((npx * npy, 2), -1, np.int32)
    lib.pixels(npx, npy, xy.ctypes.data_as(C.c_void_p))
    return xy


@pytest.mark.parametrize("npx,npy", [(1, 1), (1, 300), (300, 1), (2, 3), (7, 9), (8, 8), (16, 16), (17, 17), (15, 33),
                                     (33, 15), (70, 3), (3, 70), (64, 64), (100, 172), (16384, 2), (1, 16384)])
def test_image_order_takes_every_pixel_once(lib, npx, npy):
    xy = pixels(lib, npx, npy)
    assert xy.min() >= 0 and xy[:, 0].max() == npx - 1 and xy[:, 1].max() == npy - 1
    assert np.array_equal(np.sort(xy[:, 0] + npx * xy[:, 1]), np.arange(npx * npy))


def test_image_order_of_whole_tiles(lib):
    xy = pixels(lib, 48, 32)
    for size, side in ((64, 8), (256, 16)):
        for t in xy.reshape(-1, size, 2):
            assert (t.max(0) - t.min(0) == side - 1).all() and (t.min(0) % side == 0).all()


def test_image_wavefronts_have_pixels(lib):
    """No image shape leaves more than 0.3 of its wavefronts' lanes idle."""
    for npix in [*range(1, 700), 17 * 17, 3 * 70, 16384, 100 * 172]:
        for maps in (1, 7, 64, 4096):
            waves = lib.waves(npix, maps)
            assert 64 * waves >= npix * maps
            assert 0.7 * 64 * (waves - 1) <= npix * maps, (npix, maps)


def test_packets_per_wavefront(lib):
    """A share that covers the run with the blocks that run at a time, and no more
    than a packet per wavefront above it."""
    for total in (1, 2, 63, 3072, 3073, 20000, 196607, 196608, 300000, 10 ** 9):
        for blocks, waves in ((256, 4), (768, 4), (768, 1), (2048, 2)):
            n = lib.lanes(total, blocks, waves)
            assert 1 <= n <= 64
            assert n == 64 or (n - 1) * blocks * waves < total <= n * blocks * waves
