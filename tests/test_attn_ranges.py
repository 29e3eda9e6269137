"""The rule that cuts a cache into ranges (csrc/attn_ranges.h), compiled for the host: how many ranges
it gives, on what that depends, and that the cases the GPU tests run are the ones they are meant to be."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2502_06888_amd", "csrc")

# (head_dim, q heads, kv heads, sequences and cached positions per batch, caches on the host), and the
# ranges each batch's caches are cut into
CUT = [
    (128, 6, 1, (1,), (4000,), False, (126,)),             # the last range is the new position alone
    (128, 2, 1, (4,), (1856,), False, (59,)),              # the same with loads not requested ahead
    (64, 20, 4, (3,), (2047,), True, (32,)),               # whole loop passes, caches streamed
    (32, 32, 4, (60,), (2999,), False, (2,)),              # two ranges
    (32, 4, 4, (1, 2, 1), (1500, 0, 255), False, (12, 1, 1)),  # cut and whole caches in one launch
    (128, 8, 1, (2, 3), (900, 3000), False, (29, 94)),     # two numbers of ranges in one launch
    (128, 14, 2, (5, 2), (321, 350), True, (11, 11)),
]


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    d = tmp_path_factory.mktemp("ranges")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text('#include "attn_ranges.h"\n'
                   'extern "C" int ranges(int len, long pairs, int G, int hd, int most) { return kattn::attn_ranges(len, pairs, G, hd, most); }\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(so), str(src)], check=True)
    f = C.CDLL(str(so)).ranges
    f.argtypes = [C.c_int, C.c_long, C.c_int, C.c_int, C.c_int]
    return lambda length, pairs, G, hd, most=1 << 20: f(length, pairs, G, hd, most)


def test_gpu_cases_are_cut_as_they_say(ranges):
    for hd, hq, hkv, seqs, pos, on_host, want in CUT:
        # batches on the device share a launch; streamed ones have one each
        rows = [s if on_host else sum(seqs) for s in seqs]
        got = tuple(ranges(p + 1, r * hkv, hq // hkv, hd) for p, r in zip(pos, rows))
        assert got == want, (hd, hq, hkv, seqs, pos)
    assert ranges(322, 14, 2, 128) == 11 and ranges(31, 14, 2, 128) == 1    # ranges of 30 positions; whole
    assert ranges(901, 26, 8, 128) > 1


@pytest.mark.parametrize("hd", [32, 64, 128])
@pytest.mark.parametrize("G", [1, 4, 5, 8])
def test_rule_is_bounded_and_no_range_is_shorter_than_a_pass(ranges, hd, G):
    step = 4 * (512 // hd) * 2
    for pairs in (1, 3, 8, 32, 200, 511, 1023, 1025, 4096):
        for length in (1, 2, step, step + 1, 2 * step, 500, 1024, 4001, 16001, 100000):
            n = ranges(length, pairs, G, hd)
            slots = 256 * (4 if G <= 4 else 3 if G <= 6 else 2)
            assert 1 <= n <= max(1, -(-length // step)) and (n == 1 or n * pairs <= 2 * slots)
            for most in (1, 2, 5):
                assert 1 <= ranges(length, pairs, G, hd, most) <= most
    assert ranges(1 << 20, 1, G, hd) > 1 and ranges(step, 1, G, hd) == 1 and ranges(513, 4096, G, hd) == 1
