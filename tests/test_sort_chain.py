"""The look-back of the radix sort's chained scan, compiled for the host: sums over the tiles before one whatever order their
states arrive in, an end to every wait, and places in range whatever the states hold."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_02703_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "chain.h"
using namespace gsk;

int main() {
  std::mt19937 rng(1);
  int bad = 0;
  // states that arrive while they are waited for, as counts or as whole sums (tile 0's is whole)
  for (int round = 0; round < 2000; ++round) {
    const int tiles = 1 + rng() % 40;
    std::vector<uint32_t> count(tiles), state(tiles), final(tiles);
    uint32_t sum = 0;
    for (int t = 0; t < tiles; ++t) {
      count[t] = rng() % 3 ? rng() % 8192 : 0;
      sum += count[t];
      final[t] = t == 0 || rng() % 4 == 0 ? kWhole | sum : count[t] + 1;
      state[t] = rng() % 2 ? final[t] : 0;
    }
    auto load = [&](int j) {
      if (j < 0 || j >= tiles) { ++bad; return 0u; }
      const uint32_t v = state[j];
      const int t = rng() % tiles;
      state[t] = final[t];
      return v;
    };
    if (keys_before<8>(tiles, 1 << 20, load) != sum) ++bad;
  }
  printf("sums %d\n", bad);
  // states taken away, never whole, or of another sort: every wait ends, every load is of a tile before this one
  for (int kind = 0; kind < 4; ++kind)
    for (int tiles : {1, 2, 7, 8, 9, 40}) {
      long loads = 0;
      auto load = [&](int j) {
        if (j < 0 || j >= tiles) ++bad;
        ++loads;
        return kind == 0 ? 0u : kind == 1 ? 1u + j : kind == 2 ? (j % 3 ? 5u : 0u) : (loads % 7 ? 0u : (uint32_t)rng() & ~kWhole);
      };
      keys_before<8>(tiles, 1000, load);
      if (loads > 8000) ++bad;
    }
  printf("waits %d\n", bad);
  for (uint32_t n : {1u, 8193u, 0x7fffffffu})
    for (int i = 0; i < 1000; ++i) {
      const uint32_t first = i % 3 ? rng() : rng() % n;
      const int p = rng() % 8192;
      const uint32_t at = key_place(first, p, n);
      if (at >= n) ++bad;
      if ((uint64_t)first + p < n && at != first + p) ++bad;
    }
  printf("places %d\n", bad);
  return bad != 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("chain")
    (d / "chain.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(d / "chain.cpp"), "-o", str(d / "chain")],
                   check=True)
    return str(d / "chain")


def test_the_look_back_sums_ends_and_stays_in_range(program):
    r = subprocess.run([program], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
