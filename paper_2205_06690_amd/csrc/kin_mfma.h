// The kinetic step in FP64 as block matrix products on the matrix cores:
// geometry, host table and launchers.
#pragma once
#include "prop_kernels.h"

#include <cstddef>
#include <vector>

namespace bse {

// A line of N = R J points, x = j + J s: a DFT over s (R points, in a lane's
// registers), one J x J matrix per residue m < R, the inverse DFT over m.
template <int N> struct KinGeo;
template <> struct KinGeo<16> { static constexpr int R = 1, J = 16; };
template <> struct KinGeo<24> { static constexpr int R = 2, J = 12; };
template <> struct KinGeo<32> { static constexpr int R = 2, J = 16; };
template <> struct KinGeo<48> { static constexpr int R = 3, J = 16; };
template <> struct KinGeo<64> { static constexpr int R = 4, J = 16; };

// grids whose plane pass, and whose x pass, run so
inline bool kin_yz_grid(int n) { return n == 16 || n == 24 || n == 32 || n == 48 || n == 64; }
inline bool kin_x_grid(int n) { return n == 16 || n == 24 || n == 32; }

// the table for exp(-i k^2 dt / 2) on n points of spacing h: [R][J / 4][64
// lanes] complex, the A operands of the 16 x 16 x 4 matrix instruction
void kin_table(int n, double h, double dt, std::vector<double>& out);

// groups of orbitals whose densities the plane pass sums apart, and the parts
// it leaves for B pairs beside busy planes of other systems (1, or one per
// group where the planes are few)
constexpr int kin_yz_groups(int n) { return n <= 32 ? 5 : 2; }
int kin_yz_parts(int n, int B, int busy);

void configure_kin(int n);
// as launch_prop_x, launch_prop_yz
hipError_t launch_kin_x(int n, const PropXArgs<double>& a, int F, hipStream_t st, int tc, const LaunchEvents* ev);
hipError_t launch_kin_yz(int n, const PropYZArgs<double>& a, int nb, hipStream_t st, int nt, const LaunchEvents* ev);

}  // namespace bse
