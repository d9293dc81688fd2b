// Host build of the read-back's row placement (put_row of csrc/sph_kernels.h)
// for a CPU test: rows and features of a random order come out in the caller's
// order, and ids past the job's count, as a lost scan tile may leave them,
// write nothing outside the rows (guard words on both sides).  Prints "ok".
#include "../paper_2003_01061_amd/csrc/sph_mesh.hip"

#include <cstdio>
#include <random>

template <int D>
static bool run(std::mt19937_64 &rng, int n, bool broken, int rows, int features) {
  const size_t body = (rows ? 24 * (size_t)n : 0) + (features ? 4 * (size_t)n : 0), guard = 1024;
  std::vector<char> buf(body + 2 * guard, 0x5a);
  std::vector<uint32_t> id(n);
  for (int k = 0; k < n; ++k) id[k] = (uint32_t)k;
  std::shuffle(id.begin(), id.end(), rng);
  if (broken)
    for (int k = 0; k < n; k += 3) id[k] = k % 2 ? (uint32_t)n + (uint32_t)(rng() % 40) : (uint32_t)rng();
  std::vector<char> seen(n, 0);
  for (int k = 0; k < n; ++k) {
    const double4 x = make_double4(id[k] + 0.25, id[k] + 0.5, id[k] + 0.75, 1.0);
    put_row<D>(buf.data() + guard, n, id[k], x, (int)(id[k] % 7) + 3 * MAXF, rows, features);
    if (id[k] < (uint32_t)n) seen[id[k]] = 1;
  }
  for (size_t b = 0; b < guard; ++b)
    if (buf[b] != 0x5a || buf[guard + body + b] != 0x5a) return false;
  const double *r = reinterpret_cast<const double *>(buf.data() + guard);
  const int32_t *f = reinterpret_cast<const int32_t *>(buf.data() + guard + (rows ? 24 * (size_t)n : 0));
  for (int k = 0; k < n; ++k) {
    if (!seen[k]) continue;
    if (rows && (r[3 * k] != k + 0.25 || r[3 * k + 1] != k + 0.5 || r[3 * k + 2] != (D == 3 ? k + 0.75 : 0.0)))
      return false;
    if (features && f[k] != k % 7) return false;
  }
  return true;
}

int main() {
  std::mt19937_64 rng(29);
  for (int n : {1, 2, 67, 1000})
    for (int what = 0; what < 4; ++what)
      for (int broken = 0; broken < 2; ++broken)
        if (!run<2>(rng, n, broken, what & 1, what >> 1) || !run<3>(rng, n, broken, what & 1, what >> 1)) {
          std::printf("n %d what %d broken %d\n", n, what, broken);
          return 1;
        }
  std::printf("ok\n");
  return 0;
}
