"""The rules of the expert kernels' tiles (csrc/tile_rules.h), compiled for the host: which launches take short
tiles, and that the tile tables hold what the plan cuts."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2502_06888_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text('#include "tile_rules.h"\n'
                   'extern "C" int low(long n, int k, int E, int S, int f, int q4) { return kmoe::short_tiles(n, k, E, S, f, q4 != 0); }\n'
                   'extern "C" int most(int rowblks, int E, int S, int tokens, int q4) { return kmoe::max_tiles_for(rowblks, E, S, tokens, q4 != 0); }\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(so), str(src)], check=True)
    lib = C.CDLL(str(so))
    lib.low.argtypes = [C.c_long] + [C.c_int] * 5
    return lib


# (experts, shared, top-k, f, 4 bits) and the last number of tokens with short tiles (0: never)
LAST = [(8, 0, 2, 14336, 1, 192), (128, 0, 2, 1536, 1, 3072),
        (8, 1, 2, 14336, 1, 256), (8, 2, 2, 14336, 1, 256), (8, 4, 2, 4096, 1, 256), (15, 1, 2, 4096, 1, 480),
        (16, 1, 2, 4096, 1, 768), (16, 2, 4, 4096, 1, 384), (64, 2, 6, 1408, 1, 1024), (128, 1, 2, 1536, 1, 6144),
        (160, 2, 6, 1408, 1, 2560), (16, 0, 2, 512, 1, 0),
        (64, 2, 6, 1408, 0, 512), (64, 0, 6, 1408, 0, 0), (16, 1, 4, 1792, 0, 0)]


@pytest.mark.parametrize("E,S,k,f,q4,last", LAST)
def test_where_short_tiles_end(rules, E, S, k, f, q4, last):
    took = [n for n in range(1, 8000) if rules.low(n, k, E, S, f, q4)]
    assert (took[-1] if took else 0) == last


def test_tile_tables_hold_every_plan(rules):
    """Assignments dealt out to few experts, evenly, or one row past a block each: the tiles of a plan at either
    height it may take fit the table of a context of any larger capacity."""
    g = np.random.Generator(np.random.PCG64(11))
    for _ in range(3000):
        E, S, q4 = int(g.integers(1, 257)), int(g.integers(0, 9)), int(g.integers(0, 2))
        k = int(g.integers(1, min(E, 8) + 1))
        n = int(2 ** g.uniform(0, 14))
        f = 64 * int(g.integers(1, 200))
        room = n + int(g.integers(0, 3)) * int(g.integers(0, 3000))
        counts = np.bincount(g.integers(0, int(g.integers(1, E + 1)), size=n * k), minlength=E)
        tall = 2 if rules.low(n, k, E, S, f, q4) else 8
        blocks = -(-counts // 32)
        tiles = int((-(-blocks // tall)).sum()) + S * -(-(-(-n // 32)) // tall)
        assert tiles <= rules.most(-(-room * k // 32) + E, E, S, room, q4), (E, S, k, n, room, q4)
