"""The tiled attention kernel's choice of workgroup geometry (csrc/attn_geom.h,
plain C++, compiled here with g++): what a call's grid costs in rounds over the
CUs, counted from the printed rows and LDS of each geometry."""
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_11267_amd", "csrc")
SMALL, NORMAL, BIG, QUARTER, PAIR = range(5)
CUS, LDS = 256, 160 * 1024

PROGRAM = r"""
#include <cstdio>
#include <utility>
#include "attn_geom.h"
using namespace sdattn;
template <int D, int G> void print() {
    using T = Geom<D, G>;
    printf("geom %d %d %d %d %d %d %d\n", D, G, (int)T::kFits, T::kBQ, T::kWaves, T::kLdsBytes, T::kWavesPerSimd);
}
template <int... Ds> void print_all(std::integer_sequence<int, Ds...>) {
    ((print<32 + 8 * Ds, 0>(), print<32 + 8 * Ds, 1>(), print<32 + 8 * Ds, 2>(), print<32 + 8 * Ds, 3>(),
      print<32 + 8 * Ds, 4>()), ...);
}
template <int... Ds> int pick(int D, long long heads, int Lq, int Lk, std::integer_sequence<int, Ds...>) {
    int r = -1;
    ((D == 32 + 8 * Ds ? (void)(r = pick_geometry<32 + 8 * Ds>(heads, Lq, Lk)) : (void)0), ...);
    return r;
}
int main() {
    std::make_integer_sequence<int, 17> ds;
    print_all(ds);
    int D, Lq, Lk;
    long long heads;
    while (scanf("%d %lld %d %d", &D, &heads, &Lq, &Lk) == 4)
        printf("pick %d\n", pick(D, heads, Lq, Lk, ds));
}
"""


@pytest.fixture(scope="module")
def picks(tmp_path_factory):
    """({(D, geometry): (rows, waves, LDS bytes, waves per SIMD)}, [(call, geometry)])"""
    d = tmp_path_factory.mktemp("geom")
    (d / "geom.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.environ.get("GEOM_DIR", CSRC),
                    str(d / "geom.cpp"), "-o", str(d / "geom")], check=True)
    rng = random.Random(11)
    calls = [(D, h, 128, Lk) for D in (32, 40, 48, 56, 64) for Lk in (300, 1024)
             for h in (256, 257, 300, 320, 384, 448, 511, 512, 513)]           # one 128-row block a head
    calls += [(D, h, 64, 300) for D in (40, 64, 80) for h in (1, 255, 256, 257, 300, 511, 513)]
    calls += [(D, 8 * b, L, L) for D in (40, 64, 80, 160) for b in (1, 2, 3, 4, 8) for L in (200, 700, 1024, 2000, 4096)]
    calls += [(rng.choice(range(32, 168, 8)), rng.randrange(1, 700), rng.randrange(1, 5000), rng.randrange(129, 5000))
              for _ in range(400)]
    out = subprocess.run([str(d / "geom")], input="".join("%d %d %d %d\n" % c for c in calls), text=True,
                         capture_output=True, check=True).stdout.splitlines()
    geom, chosen = {}, []
    for line in out:
        w = line.split()
        if w[0] == "geom" and int(w[3]):
            geom[int(w[1]), int(w[2])] = tuple(int(x) for x in w[4:])
        elif w[0] == "pick":
            chosen.append(int(w[1]))
    assert len(chosen) == len(calls)
    both = [(c, g) for c, g in zip(calls, chosen)
            if (c[0], SMALL) in geom and (c[0], NORMAL) in geom]   # other widths take the general kernel
    assert len(both) > 300
    return geom, both


def rounds(heads, Lq, rows):
    return -(-heads * -(-Lq // rows) // CUS)


def test_choice_fits(picks):
    geom, both = picks
    for (D, heads, Lq, Lk), g in both:
        assert (D, g) in geom and geom[D, g][2] <= LDS


def test_rows_past_the_sequence_buy_no_rounds(picks):
    """More rows a workgroup only where that saves rounds."""
    geom, both = picks
    for (D, heads, Lq, Lk), g in both:
        rows = geom[D, g][0]
        if rows > 64:
            assert rounds(heads, Lq, rows) < rounds(heads, Lq, rows // 2), (D, heads, Lq, Lk, g)


def test_smaller_blocks_add_no_rounds(picks):
    """64 rows never in more rounds than 128."""
    geom, both = picks
    for (D, heads, Lq, Lk), g in both:
        if geom[D, g][0] == 64:
            assert rounds(heads, Lq, 64) <= rounds(heads, Lq, 128), (D, heads, Lq, Lk, g)


def test_past_one_round_a_cu_has_eight_waves(picks):
    """Two waves for every SIMD wherever there are workgroups enough."""
    geom, both = picks
    for (D, heads, Lq, Lk), g in both:
        rows, waves, lds, _ = geom[D, g]
        if rounds(heads, Lq, rows) > 1 and rows > 64:
            assert LDS // lds * waves >= 8, (D, heads, Lq, Lk, g)


def test_register_budget_follows_the_waves_on_a_cu(picks):
    """512 registers where the LDS leaves each SIMD one wave, 256 from two on."""
    geom, _ = picks
    for key, (rows, waves, lds, per_simd) in geom.items():
        on_cu = LDS // lds * waves
        if on_cu <= 4 or on_cu >= 8:
            assert per_simd == (1 if on_cu <= 4 else 2), key
