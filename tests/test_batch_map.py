"""Workgroup numbering of one-launch batched calls whose units take two
workgroups each (csrc/hh_batch_map.h), compiled for the host."""
import os
import subprocess

import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                      "paper_1811_01277_amd", "csrc", "hh_batch_map.h")
MAIN = """
#include "%s"
#include <cstdio>
#include <cstdlib>
int main(int, char** v) {
  std::printf("%%d\\n", ehh::kDies);
  for (int id = 0; id < std::atoi(v[1]); ++id) {
    const ehh::HalfUnit h = ehh::half_unit(id, std::atoi(v[2]) != 0);
    std::printf("%%d %%d\\n", h.entry, h.half);
  }
}
"""


@pytest.fixture(scope="module")
def half_unit(tmp_path_factory):
    d = tmp_path_factory.mktemp("map")
    src, exe = d / "map.cpp", d / "map"
    src.write_text(MAIN % HEADER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", str(src), "-o", str(exe)], check=True)

    def run(ids, mapped):
        out = subprocess.run([str(exe), str(ids), str(int(mapped))], check=True,
                             capture_output=True, text=True).stdout.splitlines()
        return int(out[0]), [tuple(int(x) for x in line.split()) for line in out[1:]]
    return run


@pytest.mark.parametrize("entries", [8, 64, 1016])
def test_both_halves_of_a_mapped_unit_stay_on_its_die(half_unit, entries):
    dies, got = half_unit(2 * entries, True)
    assert entries % dies == 0
    assert sorted(got) == [(e, h) for e in range(entries) for h in (0, 1)]
    for i, (entry, _) in enumerate(got):
        assert i % dies == entry % dies
    # entries start in the map's order, which is that of decreasing work
    assert all(e // dies == i // (2 * dies) for i, (e, _) in enumerate(got))


@pytest.mark.parametrize("entries", [1, 2, 7, 8, 33])
def test_unmapped_units_are_numbered_in_order(half_unit, entries):
    _, got = half_unit(2 * entries, False)
    assert got == [(e, h) for e in range(entries) for h in (0, 1)]
