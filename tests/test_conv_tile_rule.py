"""The tile rule of the convolutions (csrc/kp_conv_rule.hpp), compiled on its own:
test_gpu_conv_tiles.py repeats it to know which tiles its networks reach, so its
copy has to agree with the rule, and the rule has to give every tile for them,
forward and for input gradients."""
import ctypes as C
import os
import subprocess

import pytest

import test_gpu_conv_tiles as T

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_01283_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    tmp = str(tmp_path_factory.mktemp("tile"))
    src, lib = os.path.join(tmp, "tile.cpp"), os.path.join(tmp, "libtile.so")
    with open(src, "w") as f:
        f.write('#include "kp_conv_rule.hpp"\nextern "C" void tile(int b, int h, int w, int ci, int co, int* out) {\n'
                '  kp::dn::conv_tile_shape(b, h, w, ci, co, out[0], out[1]);\n}\n')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib],
                   check=True)
    dll = C.CDLL(lib)

    def tile(b, h, w, ci, co):
        out = (C.c_int * 2)()
        dll.tile(b, h, w, ci, co, out)
        return out[0], out[1]
    return tile


def test_the_copy_is_the_rule(rule):
    picks = set()
    for b in (1, 2, 5, 8):
        for h, w in ((32, 32), (46, 62), (100, 172), (134, 102), (256, 256), (2, 8192), (8192, 2)):
            for ci in (8, 16, 48, 80, 144, 192, 512, 1024):
                for co in (16, 32, 48, 64, 80, 96, 112, 128, 192, 512):
                    picks.add(rule(b, h, w, ci, co))
                    assert rule(b, h, w, ci, co) == T.tile(b, h, w, ci, co), (b, h, w, ci, co)
    assert {n for _, n in picks} == {1, 2, 3, 4} and {r for r, _ in picks} == {32, 16, 8}


def test_the_networks_reach_every_tile(rule, monkeypatch):
    monkeypatch.setattr(T, "tile", rule)
    every = {(r, n) for r in (32, 16, 8) for n in (1, 2, 3, 4)}
    for k, what in enumerate(("forward", "input gradients")):
        assert set().union(*(T.tiles(w, *s)[k] for w, s in T.NETS)) == every, what
