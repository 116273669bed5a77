"""The K ranges of a layer's three gradient products (csrc/gemm_plan.h, plain functions of sizes), compiled for the host and asked about thousands of layers:
what is chosen lies in the room that the workspace plan gives the products' parts, and no choice that does so too is expected to be faster."""
import os
import random
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "gemm_plan.h"
using namespace lstm;
int main() {
  long frames, n_in, n; int D;
  while (scanf("%ld %ld %ld %d", &frames, &n_in, &n, &D) == 4) {
    const TileProduct p[3] = {{frames, n_in, 4 * n, 1, D}, {n_in, 4 * n, frames, D, 1}, {n, 4 * n, frames, D, 1}};      // dX, dW_x, dW_h
    int own[3], ks[3];
    size_t room = 0, used = 0;
    for (int i = 0; i < 3; ++i) {                  // the plan: what each would take by itself
      own[i] = tile_ranges(tile_count(p[i].M, p[i].N, p[i].nz), 0, tile_stages(p[i].K, p[i].nseg));
      room += tile_part_room(p[i].M, p[i].N, p[i].nz, own[i]);
    }
    const double cost = tile_ranges3(p, room, ks);
    for (int i = 0; i < 3; ++i) used += tile_part_room(p[i].M, p[i].N, p[i].nz, ks[i]);
    int none[3];
    printf("%zu %zu %d %d %d %.6f %.6f\n", used, room, ks[0], ks[1], ks[2], cost, tile_ranges3(p, 0, none));
  }
}
"""


def test_gradient_products_ranges_fit_their_room(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_1805_05225_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    rng = random.Random(1)
    layers = [(1622, 1733, 833, 2), (2076, 1304, 931, 2), (1680, 1616, 808, 2), (64, 8, 136, 1), (2037, 660, 330, 2), (1, 1, 129, 1)]
    for _ in range(20000):
        layers.append((int(2 ** rng.uniform(0, 14)), int(2 ** rng.uniform(3, 11.5)), int(2 ** rng.uniform(7, 11)), rng.choice((1, 2))))
    out = subprocess.run([str(exe)], input="\n".join("%d %d %d %d" % l for l in layers), capture_output=True, text=True, check=True).stdout.split("\n")
    cut = 0
    for layer, line in zip(layers, out):
        used, room, k0, k1, k2 = map(int, line.split()[:5])
        cost, whole = map(float, line.split()[5:])
        assert used <= room, (layer, line)
        assert min(k0, k1, k2) >= 1 and max(k0, k1, k2) <= 16 and cost <= whole, (layer, line)
        cut += max(k0, k1, k2) > 1
    assert cut > len(layers) // 4                # (the room does not do away with ranges)
