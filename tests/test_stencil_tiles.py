"""Halo slots of the stencil tiles: every shape that the library admits, in
every vector width that it is run with, fits the slots of the variant that the
launch picks (the header that the kernels are built from, compiled for the
host)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_23612_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "stencil_tile.h"
using namespace hcu;
template <int VX>
int check(int R, int n1, int TX, int TYt, int RY, int* shapes) {
  if (halo_slots(n1, TX, TYt, TYt * RY, R) > kHaloSlots) return 0;   // not admitted
  ++*shapes;
  // vectors of the tile's halo, one by one: 2 R rows of the tile, and in x whole vectors of margin
  const int RM = (R + VX - 1) / VX * VX;
  int n = 0;
  for (int row = -R; row < TYt * RY + R; ++row)
    for (int x = -RM; x < TX + RM; x += VX) {
      const bool in_x = x >= 0 && x < TX, in_y = row >= 0 && row < TYt * RY;
      if (in_x != in_y && !(in_y && TX == n1 && n1 >= RM)) ++n;
    }
  const int per = halo_vectors(n1, TX, TYt, TYt * RY, R, VX);
  const int have = per <= kSlots<VX, true> ? kSlots<VX, true> : kSlots<VX, false>;
  if (n <= have * TX * TYt) return 0;
  std::printf("order %d, tile %d x %d, %d points of %d: %d vectors, %d slots of %d threads\n", 2 * R, TX, TYt, RY, VX, n,
              have, TX * TYt);
  return 1;
}
int main() {
  int bad = 0, shapes = 0;
  for (int R = 1; R <= 6; ++R)
    for (int TX = 1; TX <= 1024; ++TX)
      for (int TYt = 1; TX * TYt <= 1024; ++TYt)
        for (int RY = 1; RY <= 4; RY *= 2)
          for (int wide = 0; wide < 2; ++wide) {
            const int n1 = TX + 4 * wide;
            bad += check<1>(R, n1, TX, TYt, RY, &shapes);
            if (R != 4 && R != 6) continue;   // orders built with vectors
            if (RY >= 2 && TX % 2 == 0) bad += check<2>(R, n1, TX, TYt, RY, &shapes);
            if (RY >= 4 && TX % 4 == 0) bad += check<4>(R, n1, TX, TYt, RY, &shapes);
          }
  std::printf("%d shapes\n", shapes);
  return bad != 0 || shapes < 1000;
}
"""


def test_every_admitted_tile_fits_its_halo_slots(tmp_path):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
