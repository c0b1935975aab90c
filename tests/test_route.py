"""Which pipeline counts a graph (csrc/route.h, plain C++ compiled here): both
sides of every line of the rules, and the graphs of the GPU tests that name a
pipeline."""
import os
import subprocess

import numpy as np
import pytest

import test_gpu_one_sided as one_sided

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_17707_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "route.h"
int main() {
    using namespace bbc;
    RouteInput r{};
    long long nu, nv, m;
    int au, pv, bl, kn, dup;
    while (std::scanf("%lld %lld %lld %d %d %d %d %d", &nu, &nv, &m, &au, &pv, &bl, &kn, &dup) == 8) {
        if (pv == 2) {  // au: words of a band
            const int lw = band_log(au, std::max(nu, nv));
            std::printf("index %d %lld\n", lw, (long long)index_words(nu, nv, m, lw));
            continue;
        }
        MatrixShape s{};
        r = RouteInput{nu, nv, m, au != 0, pv != 0, bl != 0, kn != 0, dup != 0, 256};
        const Route x = choose_route(r, &s);
        std::printf("%s %d %d %d\n", x == Route::kMatrix ? "matrix" : x == Route::kTwoSided ? "two" : "one", s.tile, s.rpad,
                    s.kpad);
    }
}
"""


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src = d / "main.cpp"
    src.write_text(MAIN)
    exe = str(d / "main")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", exe, str(src)])

    def ask(n_u, n_v, m, raw=None, side="auto", per_vertex=False, blocks=False, knobs=False, dup=True):
        au = side == "u" or (side == "auto" and n_u < n_v)
        line = raw or " ".join(str(int(x)) for x in (n_u, n_v, m, au, per_vertex, blocks, knobs, dup))
        out = subprocess.run([exe], input=line + "\n", capture_output=True, text=True, check=True).stdout.split()
        if raw:
            return out
        return out[0], tuple(map(int, out[1:]))

    return ask


def bands(degrees, lw):
    """Bands of a side's ranks (ascending degree): whole bands of 2^(lw + 2),
    2^(lw + 1) and 2^lw ranks below the first rank of degree 16, 256 and 65536,
    then bands of 2^(lw - 1)."""
    end, at, n = len(degrees), 0, 0
    for k, d in enumerate((16, 256, 65536, None)):
        top = end if d is None else int(np.searchsorted(degrees, d))
        size = 1 << (lw + 2 - k)
        c = -(-(end - at) // size) if top >= end else (top - at) // size
        n += c
        at = min(at + c * size, end)
    return n


@pytest.mark.parametrize("words", [4096, 16384, 32768])
@pytest.mark.parametrize("seed", range(40))
def test_index_words(route, words, seed):
    """The band index never has more entries than it is given room for."""
    rng = np.random.default_rng(seed)
    n_a, n_b = (int(x) for x in np.exp(rng.uniform(np.log(3), np.log(300_000), 2)))
    m = int(np.exp(rng.uniform(np.log(2), np.log(3_000_000))))
    out = route(n_a, n_b, m, raw=f"{n_a} {n_b} {m} {words} 2 0 0 0")
    lw, room = map(int, out[1:])
    p = np.arange(1, n_b + 1) ** rng.uniform(0, 3)
    deg_b = np.sort(rng.multinomial(m, p / p.sum()))
    nb = bands(deg_b, lw)
    # lists of side a: random, all of one length, and as many as the entries of a band each give
    for lists in (rng.multinomial(m, np.full(n_a, 1 / n_a)), np.full(n_a, m // n_a), np.full(min(n_a, m // nb), nb),
                  np.ones(min(n_a, m), int)):
        indexed = (lists >= nb) | ((lists > 0) & (nb <= 16))
        assert (0 if nb <= 1 else int(indexed.sum()) * (nb + 1)) <= room


TOTALS = [
    # the sides' ratio: at most 8 to 1, either way
    ((80_000, 10_000, 300_000), "two"), ((80_001, 10_000, 300_000), "one"), ((10_000, 80_001, 300_000), "one"),
    # the mean degree over both sides: at most 64
    ((20_000, 20_000, 1_280_000), "two"), ((20_000, 20_000, 1_280_001), "one"),
    # the widest side, the most edges, no edge
    ((1 << 28, 1 << 26, 1_000_000), "two"), (((1 << 28) + 1, 1 << 26, 1_000_000), "one"),
    ((1 << 27, 1 << 27, 1 << 29), "two"), ((1 << 27, 1 << 27, (1 << 29) + 1), "one"), ((5, 5, 0), "one"),
    # small and dense graphs; 65,535 centres at most
    ((2000, 1000, 20_000), "matrix"), ((2, 65_535, 60_000), "matrix"), ((2, 65_536, 60_000), "one"),
    ((3000, 3000, 2_000_000), "matrix"), ((10_000, 10_000, 200_000), "two"),
]


@pytest.mark.parametrize("size,want", TOTALS)
def test_totals(route, size, want):
    assert route(*size)[0] == want
    # a knob of the walk, or no check for repeated pairs: no matrix
    walk = "two" if want == "matrix" and max(size[:2]) <= 8 * min(size[:2]) and size[2] ** 2 <= 4096 * size[0] * size[1] \
        else "one" if want == "matrix" else want
    assert route(*size, knobs=True)[0] == walk
    assert route(*size, dup=False)[0] == walk
    assert route(*size, blocks=True)[0] == "one"


PER_VERTEX = [
    ((5000, 5000, 60_000), "two"), ((5000, 5000, 59_999), "one"), ((5000, 4999, 60_000), "one"),
    ((20_000, 20_000, 1_400_000), "two"), ((20_000, 20_000, 1_400_001), "one"),
    ((32_768, 32_768, 12_000_000), "two"), ((32_767, 32_768, 12_000_000), "one"),
    ((300_000, 37_500, 1_000_000), "two"), ((300_001, 37_500, 1_000_000), "one"),
]


@pytest.mark.parametrize("size,want", PER_VERTEX)
def test_per_vertex(route, size, want):
    assert route(*size, per_vertex=True)[0] == want
    assert route(*size, per_vertex=True, knobs=True)[0] == "one"


def test_matrix_shapes(route):
    """Rows padded to the tile, columns to 64; 64-row tiles below a tile per CU."""
    assert route(65, 64, 1000, side="u") == ("matrix", (64, 128, 64))
    assert route(2816, 65, 30_000, side="u") == ("matrix", (64, 2816, 128))
    assert route(2817, 64, 30_000, side="u") == ("matrix", (128, 2944, 64))


@pytest.mark.parametrize("name", sorted(one_sided.GRAPHS))
def test_one_sided_graphs(route, name):
    g = one_sided.GRAPHS[name]()
    for side in ("u", "v"):
        assert route(g.n_u, g.n_v, g.m, side=side, knobs=True)[0] == "one"
    if name in one_sided.BY_DEFAULT:
        assert route(g.n_u, g.n_v, g.m)[0] == "one"
