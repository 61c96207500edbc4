"""The run's host-side decisions (csrc/kp_rules.hpp), compiled on their own."""
import ctypes as C
import os
import subprocess

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
size_t grow(size_t need, size_t have, size_t elem) { return grow_bytes(need, have, elem); }
}
""")
    dll.copies.argtypes = [C.c_int, z, z, z, z, z]
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
