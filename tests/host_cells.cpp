// Host build of the grouped cell scan's row ranges (cell_split and row_range
// of csrc/sph_kernels.h) for a CPU test: every cell that the FP64 ranges of the
// one-lane kernel touch is in them, for particles inside the grid, on its
// borders, and off it by up to 1e300 cells.  Prints "ok" and the number of ranges.
#include "../paper_2003_01061_amd/csrc/sph_mesh.hip"

#include <cstdio>
#include <random>

int main() {
  std::mt19937_64 rng(23);
  std::uniform_real_distribution<double> u01(0.0, 1.0);
  const double far[] = {1e3, 0x1p29, 0x1p30, 0x1p31, 0x1p31 + 7.5, 0x1p32, 1e12, 1e18, 1e300};
  long done = 0;
  for (int t = 0; t < 400000; ++t) {
    const int nc = 1 + (int)(rng() % (t % 3 ? 300 : 1u << 29));
    double u = (double)nc * (1.5 * u01(rng) - 0.25);
    if (t % 5 == 0) u = std::floor(u);                        // on a cell border
    if (t % 7 == 0) u = (t & 1 ? -1.0 : 1.0) * far[rng() % 9] * (1.0 + u01(rng));
    if (t % 49 == 0) u = (t & 1 ? -1.0 : 1.0) * far[rng() % 9];
    const double wx = t % 11 ? std::pow(10.0, 4.0 * u01(rng) - 2.0) : 0.0;
    // as k_nbr_forces
    const double top = (double)(nc - 1), w64 = wx * (1.0 + 1e-6) + 1e-7;
    double a = std::floor(u - w64), b = std::floor(u + w64);
    a = a >= 0.0 ? a : 0.0;
    b = b >= 0.0 ? b : 0.0;
    a = a < top ? a : top;
    b = b < top ? b : top;
    // as k_nbr_group, with its widening of the half chord
    int whole, t0, t1;
    float frac;
    cell_split(u, whole, frac);
    row_range(whole, frac, (float)wx * (1.0f + 2e-6f) * (1.0f + 2e-6f) + 2e-5f, nc, t0, t1);
    if (t0 < 0 || t1 >= nc || (double)t0 > a || (double)t1 < b) {
      std::printf("u %.17g half chord %.17g of %d cells: [%d, %d], want [%.0f, %.0f]\n", u, wx, nc, t0, t1, a, b);
      return 1;
    }
    ++done;
  }
  std::printf("ok %ld\n", done);
  return 0;
}
