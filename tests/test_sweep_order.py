"""CPU checks of header code that no library entry point reaches on the host: a small program over
the csrc headers, compiled for the host alone, is run by each test."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_02044_amd", "csrc")

SWEEP = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "lattice.h"
using namespace gl;
// every site once, every (layer, slot) by one block, both mappings alike
static int cover(int nz, int nt, int bs, int64_t whole, int slab) {
  Geom g;
  g.nt = nt; g.nz = nz; g.layer = (int64_t)nt * nt; g.V = g.layer * nz; g.Vp = padded_sites(g.V);
  const ColMap m = col_map(g, bs, whole, slab);
  const int slots = col_map_slots_per_layer(m);
  std::vector<char> site(g.V, 0), slot((size_t)nz * slots, 0);
  for (uint32_t b = 0; b < col_map_blocks(g, m); ++b) {
    int z;
    uint32_t sl;
    col_map_block(m, b, z, sl);
    const bool idle = z < 0 || z >= nz;
    if (!idle) {
      if (sl >= (uint32_t)slots || slot[(size_t)z * slots + sl]++) return 1;
    }
    for (int t = 0; t < bs; ++t) {
      Site x;
      uint32_t s;
      if (!col_map_site(g, m, b, t, bs, x, s)) continue;
      if (idle || x.z != z || s >= g.V || s != site_index(g, x.x, x.y, x.z) || site[s]++) return 2;
    }
  }
  for (char c : site) if (!c) return 3;
  for (char c : slot) if (!c) return 4;
  return 0;
}
int main(int, char** v) {
  if (v[1][0] == 'q') {   // quotients
    srand(1);
    for (int k = 0; k < 4000000; ++k) {
      const uint32_t d = 1 + (((uint32_t)rand() << 15 ^ rand()) & ((1u << (1 + rand() % 29)) - 1));
      uint32_t n = ((uint32_t)rand() << 15 ^ rand()) & ((1u << 29) - 1);
      if (k & 1) n = n / d * d + (k & 2 ? d - 1 : 0);
      if (n >= 1u << 29) continue;
      if (quot(n, div_by(d)) != n / d) { printf("%u / %u\n", n, d); return 1; }
    }
    return 0;
  }
  return cover(atoi(v[1]), atoi(v[2]), atoi(v[3]), atoll(v[4]), atoi(v[5]));
}
"""


def build(tmp, name, source):
    src, out = tmp / (name + ".hip"), tmp / name
    src.write_text(source)
    subprocess.run(["hipcc", "-O2", "-std=c++20", "-w", "--cuda-host-only", "-I", CSRC, str(src), "-o", str(out)],
                   check=True, capture_output=True)
    return str(out)


@pytest.fixture(scope="module")
def sweep(tmp_path_factory):
    return build(tmp_path_factory.mktemp("sweep"), "sweep", SWEEP)


def test_quotients_by_multiplication(sweep):
    assert subprocess.run([sweep, "q"]).returncode == 0


@pytest.mark.parametrize("slab", [1, 0])
@pytest.mark.parametrize("bs", [64, 256])
def test_sweep_covers_every_site_once(sweep, bs, slab):
    """Work-group -> (layer, block) at sizes with fewer layers than XCDs, several layers per XCD of
    unequal number, one band, bands of equal size and a narrower last one (150: 88 work-groups of
    256 in 30, 30, 28; 131: 68 in 34, 34), and thresholds that turn bands on for small layers."""
    sizes = [(2, 2), (3, 5), (9, 16), (17, 21), (64, 8), (1000, 3), (5, 100), (9, 100), (17, 131), (20, 150), (9, 192)]
    g = np.random.default_rng(7)
    sizes += [(int(np.exp(g.uniform(0.7, 4.5))) + 1, int(np.exp(g.uniform(0.7, 4.9))) + 1) for _ in range(20)]
    for nz, nt in sizes:
        for whole in (9216, 16384, 64):
            assert subprocess.run([sweep, str(nz), str(nt), str(bs), str(whole), str(slab)]).returncode == 0, (nz, nt, whole)
