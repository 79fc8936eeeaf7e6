// Halo of a stencil tile: what its threads stage per plane, and the slots that
// the kernels hold it in.
#pragma once

namespace hcu {

// Slots per thread.  The admitted shapes need at most kHaloSlots of single
// points; half as many serve most tiles, and each slot costs registers.  In
// vectors of VX points the halo in x is rounded up to whole vectors (6 points
// to 8 in vectors of four), so the slots are counted in vectors as well: 8 of
// one point, 4 of two and 3 of four hold every admitted shape, and whether the
// few do is seen from the vectors (halo_vectors), not from the points.
constexpr int kHaloSlots = 8;
constexpr int kHaloSlotsSmall = 4;
template <int VX, bool SMALL>
constexpr int kSlots = VX == 4 ? (SMALL ? 1 : 3) : (SMALL ? kHaloSlotsSmall : kHaloSlots) / VX;

// halo values of a plane for a tile of TX x TY points on a grid with n1 points in x
constexpr int halo_values(int n1, int TX, int TY, int R) {
  return 2 * R * TX + ((TX == n1 && n1 >= R) ? 0 : TY * 2 * R);
}
// and per thread (TX x TYt of them)
constexpr int halo_slots(int n1, int TX, int TYt, int TY, int R) {
  return (halo_values(n1, TX, TY, R) + TX * TYt - 1) / (TX * TYt);
}
// the same in vectors of vx points (the tile's TX is a multiple of vx)
constexpr int halo_vectors(int n1, int TX, int TYt, int TY, int R, int vx) {
  const int RM = (R + vx - 1) / vx * vx;
  const int n = 2 * R * (TX / vx) + ((TX == n1 && n1 >= RM) ? 0 : TY * (2 * RM / vx));
  return (n + TX * TYt - 1) / (TX * TYt);
}

}  // namespace hcu
