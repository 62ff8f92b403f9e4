// When a power of the amplification matrix counts as rank one (see
// lbm_stability.hip); shared with a host test.
#pragma once

#include "lbm_node.h"

namespace lbm {

// Small enough that its square is below the rounding of a product (2^-53)
// many times over; any such bound serves, and a tighter one only closes later
// (Fig. 2 maps, 4 x 512 x 512 points: 12.5 ms at 2^-46, 12.2 at 2^-44 and
// 2^-42, the same errors).
constexpr double RANK_TOL = 0x1p-44;

// X^2 = mu X is compared through one entry: with o that entry of X and n of
// X^2, mu = n / o, and everything is taken times |o|^2, so that no division
// is needed: |o|^2 (X^2 - mu X) = |o|^2 X^2 - (n conj(o)) X.
struct RankOne {
  double o2, n2;  // |o|^2, |n|^2
  double mr, mi;  // n conj(o)
};

LBM_HD RankOne rank_one(double ore, double oim, double nre, double nim) {
  return {ore * ore + oim * oim, nre * nre + nim * nim, nre * ore + nim * oim, nim * ore - nre * oim};
}

// The larger component of |o|^2 (X^2 - mu X) at an entry x of X, a of X^2.
LBM_HD double rank_one_gap(const RankOne& c, double xr, double xi, double ar, double ai) {
  return fmax(fabs(c.o2 * ar - (c.mr * xr - c.mi * xi)), fabs(c.o2 * ai - (c.mr * xi + c.mi * xr)));
}

// Whether the largest gap means |X^2 - mu X| < RANK_TOL |mu| |o|: of degree
// eight in X on either side, the same for every multiple of X.
LBM_HD bool rank_one_within(const RankOne& c, double gap) {
  return gap * gap < RANK_TOL * RANK_TOL * c.n2 * (c.o2 * c.o2);
}

}  // namespace lbm
