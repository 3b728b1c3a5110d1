"""The plans of the last shapes (prom_recent.h) by themselves: against a plain list in order of use, and that a network's
blocks are all found on the second pass."""
import ctypes as C
import os
import random
import subprocess

import pytest

from workloads import mobilenetv2_blocks

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KEY = C.c_int * 8


@pytest.fixture(scope="module")
def cache(tmp_path_factory):
    """(new, get): get(cache, key, value) -> (found, what was there); the value goes in if it was not found."""
    d = tmp_path_factory.mktemp("recent")
    src, lib = d / "recent.cpp", d / "recent.so"
    src.write_text('#include "prom_recent.h"\n#include <array>\n'
                   'using R = prom::Recent<std::array<int, 8>, int, 32>;\n'
                   'extern "C" R *fresh() { return new R; }\n'
                   'extern "C" int get(R *r, const std::array<int, 8> *k, int v)\n'
                   '{ bool found; int &x = r->get(*k, &found); if (!found) { x = v; return -1; } return x; }\n')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-O1",
                    "-I" + os.path.join(ROOT, "paper_2505_03254_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    so = C.CDLL(str(lib))
    so.fresh.restype = C.c_void_p
    so.get.argtypes = [C.c_void_p, C.POINTER(KEY), C.c_int]
    return so.fresh, lambda r, key, v: so.get(r, C.byref(KEY(*key)), v)


def test_against_a_list(cache):
    fresh, get = cache
    rng = random.Random(7)
    for keys in (20, 32, 33, 60):
        r, model = fresh(), []  # (key, value), the one used last at the end
        for step in range(3000):
            k = (rng.randrange(keys), 0, 0, 0, 0, 0, 0, rng.randrange(2) if keys == 60 else 0)
            at = next((i for i, (q, _) in enumerate(model) if q == k), None)
            got = get(r, k, step)
            assert got == (-1 if at is None else model[at][1]), (keys, step)
            model.append(model.pop(at) if at is not None else (k, step))
            del model[:-32]


@pytest.mark.parametrize("batches", [(1,), (8,), (128,), (8, 128)])
def test_a_network_is_planned_once(cache, batches):
    fresh, get = cache
    for prelu in (0, 1):
        r = fresh()
        shapes = [(n, b.hw_in, b.hw_in, b.cin, b.cin * b.t, b.cout, b.stride, prelu)
                  for n in batches for b in mobilenetv2_blocks() if b.t != 1]
        for i, s in enumerate(shapes):
            get(r, s, i)
        assert all(get(r, s, -5) >= 0 for _ in range(3) for s in shapes)


def test_an_empty_cache_finds_nothing(cache):
    fresh, get = cache
    assert get(fresh(), (0,) * 8, 1) == -1
