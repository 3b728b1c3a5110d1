"""Workgroups of a shared grouped-convolution launch: the host function by itself, against an exhaustive search."""
import ctypes as C
import itertools
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Layer(C.Structure):
    _fields_ = [("blocks", C.c_int), ("units", C.c_int), ("unit_cost", C.c_double)]


@pytest.fixture(scope="module")
def shares(tmp_path_factory):
    d = tmp_path_factory.mktemp("shares")
    src, lib = d / "shares.cpp", d / "shares.so"
    src.write_text('#include "prom_gconv_shares.h"\n'
                   'extern "C" void shares(const prom::GconvShareLayer *l, int n, int slots, int *w, int *s)\n'
                   '{ prom::gconv_shares(l, n, slots, w, s); }\n')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-O1",
                    "-I" + os.path.join(ROOT, "paper_2505_03254_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    f = C.CDLL(str(lib)).shares

    def call(layers, slots):
        n = len(layers)
        w, s = (C.c_int * n)(), (C.c_int * n)()
        f((Layer * n)(*[Layer(*l) for l in layers]), n, slots, w, s)
        return list(w), list(s)
    return call


def _check(layers, slots, w, s):
    for (blocks, units, _), a, b in zip(layers, w, s):
        assert 1 <= a <= units and b in (1, 8) and a % b == 0 and (b == 1 or blocks > 1)
    return sum(a * l[0] for a, l in zip(w, layers))


def _end(layers, w):
    return max(-(-l[1] // a) * l[2] for l, a in zip(layers, w))


@pytest.mark.parametrize("seed", range(4))
def test_no_allocation_ends_sooner(shares, seed):
    rng = random.Random(seed)
    for _ in range(60):
        layers = [(1, rng.randint(1, 12), rng.choice((2.5, 3.0, 4.5))) for _ in range(rng.randint(2, 3))]
        slots = rng.randint(len(layers), 20)
        w, s = shares(layers, slots)
        assert _check(layers, slots, w, s) <= slots, (layers, slots, w)
        best = min(_end(layers, t) for t in itertools.product(*[range(1, l[1] + 1) for l in layers]) if sum(t) <= slots)
        assert _end(layers, w) <= best * 1.001, (layers, slots, w, best)
        # nothing is left that a layer could still take
        left = slots - sum(w)
        assert left == 0 or all(a == l[1] for a, l in zip(w, layers)), (layers, slots, w)


@pytest.mark.parametrize("layers,slots", [
    ([(1, 1, 2.5), (1, 1, 2.5)], 512),                            # fewer units than workgroups
    ([(64, 1000000, 4.0)] * 24, 512),                             # one workgroup per channel block does not fit
    ([(40, 8, 2.5), (40, 9, 2.5)], 512),                          # no room for a multiple of 8
    ([(2, 2000000000, 2.5), (1, 3, 30.0)], 512),                  # units near the largest int
    ([(3, 7, 2.5), (2, 8, 2.5), (2, 12, 2.5), (5, 100, 6.0)], 512),
    ([(1, 100, 2.5)] * 22, 512),
])
def test_edges(shares, layers, slots):
    w, s = shares(layers, slots)
    used = _check(layers, slots, w, s)
    assert used <= max(slots, sum(l[0] for l in layers)), (w, s)
