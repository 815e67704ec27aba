"""The arithmetic of the rules that choose a method (csrc/rips_rules.hpp is
plain C++), compiled and run on the CPU."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def run(tmp_path, body):
    src = tmp_path / "rules.cpp"
    src.write_text('#include <cmath>\n#include <cstdio>\n#include <initializer_list>\n#include "rips_rules.hpp"\n'
                   "using namespace rips;\nint main() {\n" + body + "\n}\n")
    exe = str(tmp_path / "rules")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_1908_02518_amd", "csrc"), str(src),
                    "-o", exe], check=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()


def test_triangles_are_counted_in_64_bits(tmp_path):
    """One cluster of 2955 to 3014 points has 2^32 triangles and fewer than
    2^28 more: counted in 32 bits they seem to fit."""
    got = run(tmp_path, """
    for (uint64_t k : {1173ull, 1174ull, 2954ull, 2955ull, 3014ull, 65535ull}) {
        uint64_t n = 0; // edge by edge, as they are counted
        for (uint64_t i = 2; i < k; ++i) n += i * (i - 1) / 2;
        printf("%d %d ", (int)owned_fit(n), (int)((uint32_t)n <= (1u << 28)));
    }
    printf("%d %d", (int)owned_fit(1ull << 28), (int)owned_fit((1ull << 28) + 1));""")
    fits = [int(x) for x in got[0:12:2]]
    wrapped = [int(x) for x in got[1:12:2]]
    assert fits == [1, 0, 0, 0, 0, 0]
    assert wrapped[3:5] == [1, 1]  # what a count of 32 bits would say
    assert got[12:] == ["1", "0"]


def test_count_of_pairs_fits_its_type(tmp_path):
    """However many there are: every wave of the largest grid ends with its
    first append past the capacity."""
    got = run(tmp_path, 'printf("%lld", (long long)most_pairs(kMostPairs, 16384 * 4));')
    assert int(got[0]) == (1 << 21) + 65536 * 64 < 2 ** 31


def test_sweep_flags_outside_the_two_bits_are_refused():
    import paper_1908_02518_amd as rips
    assert rips.lib().rips_set_sweep(-1) == -1  # before the device is touched
    assert rips.lib().rips_set_sweep(4) == -1
    assert rips.lib().rips_get_sweep(None) == -1


def test_sizes_of_clouds_swept_whole(tmp_path):
    got = run(tmp_path, """
    for (int d : {0, 1, 2})
        for (bool dense : {false, true})
            for (uint32_t p : {2u, 3u, 65521u}) printf("%d ", whole_most(d, dense, p));""")
    assert [int(x) for x in got] == [128] * 6 + [256, 128, 128, 1024, 200, 200] + [0] * 6


def test_classes_of_a_cloud_swept_whole(tmp_path):
    got = run(tmp_path, """
    for (int n : {2, 127, 128, 1024}) printf("%d %d ", whole_classes(n, 2), whole_classes(n, 3));""")
    assert [int(x) for x in got] == [256, 220, 256, 220, 256, 220, 2048, 220]


def test_clouds_whose_dimension_1_is_swept_in_chunks(tmp_path):
    """By the mean degree, and by its mean seen from an edge; the cluster of
    2955 among 44,000 points of no edge is out by the latter."""
    got = run(tmp_path, """
    auto even = [](int64_t n, int64_t d, uint32_t p) { return (int)chunks_pay(n, n * d / 2, (uint64_t)(n * d * d), p); };
    for (uint32_t p : {2u, 3u})
        for (int64_t d : {31, 32, 110, 111, 200, 201, 4000}) printf("%d ", even(10000, d, p));
    // half the points of degree a, half of degree b
    auto two = [](int64_t a, int64_t b) { return (int)chunks_pay(1000, 250 * (a + b), (uint64_t)(500 * (a * a + b * b)), 2); };
    printf("%d %d %d ", two(100, 100), two(146, 54), two(148, 52));
    printf("%d ", (int)chunks_pay(44000, 2955ll * 2954 / 2, 2955ull * 2954 * 2954, 2));
    printf("%d %d", (int)chunks_pay(65535, 65535ll * 100, 65535ull * 200 * 200, 2), (int)chunks_pay(65535, 0, 0, 2));""")
    assert got == "0 1 1 1 1 0 0  0 1 1 0 0 0 0  1 1 0  0  1 0".split()


def test_batches_that_are_swept(tmp_path):
    got = run(tmp_path, """
    for (uint32_t p : {2u, 3u})
        for (int n : {1, 128, 129, 2048})
            for (int m : {1, 128, 129, 100000}) printf("%d ", (int)batch_swept(n, m, p));""")
    assert [int(x) for x in got] == [1] * 8 + [1, 1, 0, 0] * 2 + [0] * 16


def test_clouds_whose_dimension_2_is_swept_by_blocks(tmp_path):
    """By the triangles, by how many an edge has, and by evenness."""
    got = run(tmp_path, """
    auto even = [](int64_t n, int64_t d, int64_t t) { return (int)blocks_pay(n, n * d / 2, (uint64_t)(n * d * d), t); };
    printf("%d %d ", even(100, 20, 12287), even(100, 20, 12288));
    printf("%d %d ", even(2000, 50, 249999), even(2000, 50, 250000));
    printf("%d %d ", (int)blocks_pay(1000, 50000, 12200000, 1 << 20), (int)blocks_pay(1000, 50000, 12200001, 1 << 20));
    for (int64_t n : {42, 43, 44}) printf("%d ", even(n, n - 1, n * (n - 1) * (n - 2) / 6));
    printf("%d", even(65535, 65534, 46907926681605ll));""")
    assert [int(x) for x in got] == [0, 1, 0, 1, 1, 0, 0, 1, 1, 1]
