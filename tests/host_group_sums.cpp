// Host build of the pressure sums of the kernels with several lanes per particle
// (group_sums of csrc/sph_kernels.h), a lane at a time, for a CPU test under
// sanitizers: on random neighbourhoods with boundary entries of every normal
// mode (constant, stored, and the pair normals of 3D patches at curves and
// vertices), lists of 0 to 61 entries read from the ring or from memory, split
// over 1, 2, 4 and 8 lanes, the lanes' sums add up to the sums written out below
// in long double from the equations; and one lane that adds as four (four_sums,
// 2D) gets the four lanes' sums bit for bit.
//
// Bar: a sum of n <= 62 terms of about 20 roundings each, added in another
// order, differs by at most (20 + 62) 2^-53 of the sum of the terms' magnitudes,
// below 1e-14 of it; 1e-13 is taken.  Prints "ok" and the number of sums.
#include "../paper_2003_01061_amd/csrc/sph_mesh.hip"

#include <cstdio>
#include <random>

using LD = long double;

static LD w_of(int k, LD r, LD h) {   // Wendland C2 of smoothing length h
  const LD q = r / h;
  if (!(q < 2)) return 0;
  const LD t = 1 - q / 2, pi = 3.14159265358979323846264338327950288L;
  const LD a = k == 1 ? LD(5) / 8 : k == 2 ? 7 / (4 * pi) : 21 / (16 * pi);
  return a * (k == 1 ? t * t * t * (1 + 1.5L * q) : t * t * t * t * (1 + 2 * q)) / powl(h, k);
}
static LD dw_of(int k, LD r, LD h) {   // (dW/dr) / r
  const LD q = r / h;
  if (!(q < 2)) return 0;
  const LD t = 1 - q / 2, pi = 3.14159265358979323846264338327950288L;
  const LD a = k == 1 ? LD(5) / 8 : k == 2 ? 7 / (4 * pi) : 21 / (16 * pi);
  return a * (k == 1 ? -3 * t * t : -5 * t * t * t) / powl(h, k + 2);
}

struct Problem {
  int n, i, bw;
  uint32_t cnt;
  double p0, klen, bscale;
  std::vector<double4> xh, enrm;
  std::vector<uint16_t> f;
  std::vector<BNorm> bn;
  std::vector<double> cpts;
  std::vector<uint32_t> entries, nbr, ring;
  bool pairs;
};

static double4 unit(std::mt19937_64 &rng, int D) {
  std::normal_distribution<double> g;
  double4 v = make_double4(g(rng), g(rng), D == 3 ? g(rng) : 0.0, 0.0);
  const double l = std::sqrt(v.x * v.x + v.y * v.y + v.z * v.z);
  return make_double4(v.x / l, v.y / l, v.z / l, 0.0);
}

template <int D, int K>
static Problem make(std::mt19937_64 &rng, uint32_t ring_len) {
  std::uniform_real_distribution<double> u(0.0, 1.0);
  Problem P;
  P.n = 80;
  P.i = (int)(rng() % P.n);
  P.cnt = (uint32_t)(rng() % 62);
  P.bw = (int)(rng() % 3);
  P.p0 = 0.5 + u(rng);
  P.klen = 0.75 + u(rng);
  P.bscale = 0.5 + u(rng);
  P.pairs = D == 3 && K == 2;
  const double h0 = std::pow(10.0, 2.0 * u(rng) - 2.0);
  for (int j = 0; j < P.n; ++j) {
    P.xh.push_back(make_double4(h0 * 2.0 * u(rng), h0 * 2.0 * u(rng), D == 3 ? h0 * 2.0 * u(rng) : 0.0,
                                h0 * (0.7 + 0.6 * u(rng))));
    double4 e = unit(rng, D);
    e.w = (double)(rng() % 9);   // a segment of the curve
    P.enrm.push_back(e);
    P.f.push_back((uint16_t)(3 * MAXF + rng() % MAXF));
  }
  P.xh[(P.i + 1) % P.n] = P.xh[P.i];   // a particle on top of i
  for (int q = 0; q < MAXF; ++q) {
    BNorm b{};
    b.mode = P.pairs ? (int)(rng() % 9) : (int)(rng() % 7);
    const double4 v = unit(rng, D);
    b.n[0] = v.x;
    b.n[1] = v.y;
    b.n[2] = v.z;
    P.bn.push_back(b);
  }
  for (int k = 0; k < 10; ++k)
    for (int a = 0; a < 3; ++a) P.cpts.push_back(u(rng) + k);
  const bool boundary = u(rng) < 0.7;
  for (uint32_t e = 0; e < P.cnt; ++e)
    P.entries.push_back((uint32_t)(rng() % P.n) | (boundary && u(rng) < 0.3 ? 0x80000000u : 0u));
  P.nbr.assign((size_t)((P.cnt + LB - 1) / LB) * P.n * LB + 1, 0xffffffffu);
  P.ring.assign(ring_len, 0xffffffffu);
  for (uint32_t e = 0; e < P.cnt; ++e) {
    P.nbr[((size_t)(e / LB) * P.n + P.i) * LB + e % LB] = P.entries[e];
    P.ring[e % ring_len] = P.entries[e];
  }
  return P;
}

struct Sums {
  LD v[8] = {}, mag[8] = {};   // S, gamma, Pi[3], B[3] and the terms' magnitudes
  void add(int k, LD t) {
    v[k] += t;
    mag[k] += fabsl(t);
  }
};

template <int D, int K>
static Sums reference(const Problem &P) {
  Sums r;
  const double4 xi = P.xh[P.i], ei = P.enrm[P.i];
  const LD hi = xi.w, kl = P.klen;
  r.add(0, w_of(K, 0, kl * hi));
  r.add(1, w_of(K, 0, kl * hi) * powl(hi, K));
  for (uint32_t v : P.entries) {
    const uint32_t j = v & 0x7fffffffu;
    const double4 xj = P.xh[j];
    const LD d[3] = {(LD)xi.x - xj.x, (LD)xi.y - xj.y, (LD)xi.z - xj.z}, hj = xj.w;
    const LD rr = sqrtl(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    const LD hs = powl(hi, 2 * K) + powl(hj, 2 * K), hij = kl * (hi + hj) / 2;
    r.add(0, w_of(K, rr, kl * hi));
    if (!(v >> 31)) {
      r.add(1, w_of(K, rr, kl * hi) * powl(hj, K));
      for (int a = 0; a < D; ++a) r.add(2 + a, P.p0 * hs * dw_of(K, rr, hij) * d[a]);
      continue;
    }
    LD nv[3];
    const BNorm &N = P.bn[P.f[j] % MAXF];
    if (K == D || (N.mode >= 2 && N.mode < 7)) {
      nv[0] = P.enrm[j].x, nv[1] = P.enrm[j].y, nv[2] = P.enrm[j].z;
    } else if (N.mode < 2) {
      nv[0] = N.n[0], nv[1] = N.n[1], nv[2] = N.n[2];
    } else {   // towards b in i's tangent plane, at a curve without its tangent
      LD m = 0, l = 0;
      for (int a = 0; a < 3; ++a) nv[a] = -d[a];
      m = nv[0] * ei.x + nv[1] * ei.y + nv[2] * ei.z;
      nv[0] -= m * ei.x, nv[1] -= m * ei.y, nv[2] -= m * ei.z;
      if (N.mode == 7) {
        const double *p = &P.cpts[3 * (size_t)P.enrm[j].w];
        LD t[3], tl = 0, dt = 0;
        for (int a = 0; a < 3; ++a) t[a] = (LD)p[3 + a] - p[a], tl += t[a] * t[a];
        for (int a = 0; a < 3; ++a) t[a] /= sqrtl(tl), dt += nv[a] * t[a];
        for (int a = 0; a < 3; ++a) nv[a] -= dt * t[a];
      }
      for (int a = 0; a < 3; ++a) l += nv[a] * nv[a];
      l = sqrtl(l);
      for (int a = 0; a < 3; ++a) nv[a] = l > 0 ? nv[a] / l : 0;
    }
    const LD om = (P.bw == 0 ? 1 / hj : P.bw == 1 ? powl(hj, K - 1) : 0) * P.bscale;
    for (int a = 0; a < D; ++a) r.add(5 + a, P.p0 * hs * w_of(K, rr, hij) * om * nv[a]);
  }
  return r;
}

template <int D, int K, int G>
static bool split(const Problem &P, const Sums &want, uint32_t ring_len, bool pairs_kernel) {
  Geom g{};
  g.cpts = P.cpts.data();
  Parts s{};
  s.xh = const_cast<double4 *>(P.xh.data());
  s.f = const_cast<uint16_t *>(P.f.data());
  double got[8] = {};
  for (uint32_t l = 0; l < G; ++l) {
    double S, gam, Pi[3], B[3];
    if (pairs_kernel)
      group_sums<D, K, double, false, true, 4, G>(g, s, P.enrm.data(), P.bn.data(), P.bw, P.p0, P.klen, P.bscale,
                                                  P.nbr.data(), P.n, P.i, P.cnt, P.xh[P.i], P.pairs, S, gam, Pi, B,
                                                  (LdsList)P.ring.data(), ring_len, l);
    else
      group_sums<D, K, double, false, false, 4, G>(g, s, P.enrm.data(), P.bn.data(), P.bw, P.p0, P.klen, P.bscale,
                                                   P.nbr.data(), P.n, P.i, P.cnt, P.xh[P.i], P.pairs, S, gam, Pi, B,
                                                   (LdsList)P.ring.data(), ring_len, l);
    const double t[8] = {S, gam, Pi[0], Pi[1], Pi[2], B[0], B[1], B[2]};
    for (int k = 0; k < 8; ++k) got[k] += t[k];
  }
  for (int k = 0; k < 8; ++k)
    if (!(fabsl(got[k] - want.v[k]) <= 1e-13L * want.mag[k])) {
      std::printf("%dD k %d, %d lanes, %u entries, ring %u: sum %d is %.17g, want %.17Lg (terms %.3Lg)\n", D, K, G,
                  P.cnt, ring_len, k, got[k], want.v[k], want.mag[k]);
      return false;
    }
  return true;
}

// four_sums against the four lanes of group_sums, added as group_sum adds them
template <int K>
static bool four(const Problem &P, uint32_t ring_len) {
  Geom g{};
  g.cpts = P.cpts.data();
  Parts s{};
  s.xh = const_cast<double4 *>(P.xh.data());
  s.f = const_cast<uint16_t *>(P.f.data());
  double lane[4][8];
  for (uint32_t l = 0; l < 4; ++l)
    group_sums<2, K, double, false, false, 4, 4>(g, s, P.enrm.data(), P.bn.data(), P.bw, P.p0, P.klen, P.bscale,
                                                 P.nbr.data(), P.n, P.i, P.cnt, P.xh[P.i], false, lane[l][0],
                                                 lane[l][1], lane[l] + 2, lane[l] + 5, (LdsList)P.ring.data(),
                                                 ring_len, l);
  for (int source = 0; source < 2; ++source) {   // from memory; with the list's end in the ring
    double got[8];
    four_sums<K, double, false>(s, P.enrm.data(), P.bn.data(), P.bw, P.p0, P.klen, P.bscale, P.nbr.data(), P.n, P.i,
                                P.cnt, P.xh[P.i], got[0], got[1], got + 2, got + 5,
                                source ? P.ring.data() : nullptr, ring_len, 1);
    for (int k = 0; k < 8; ++k) {
      const double want = (lane[0][k] + lane[1][k]) + (lane[2][k] + lane[3][k]);
      if (got[k] != want) {
        std::printf("k %d as four, %u entries: sum %d is %.17g, want %.17g\n", K, P.cnt, k, got[k], want);
        return false;
      }
    }
  }
  return true;
}

template <int D, int K>
static long run(std::mt19937_64 &rng, int trials) {
  long done = 0;
  for (int t = 0; t < trials; ++t) {
    const uint32_t ring_len = t % 2 ? 32 : 64;
    const Problem P = make<D, K>(rng, ring_len);
    const Sums want = reference<D, K>(P);
    // geometries without curves have no pair normals and may take the kernel without them
    const bool pk = P.pairs || t % 3 == 0;
    if (!split<D, K, 1>(P, want, ring_len, pk) || !split<D, K, 2>(P, want, ring_len, pk) ||
        !split<D, K, 4>(P, want, ring_len, pk) || !split<D, K, 8>(P, want, ring_len, pk))
      return -1;
    if constexpr (D == 2)
      if (!four<K>(P, ring_len)) return -1;
    done += 4;
  }
  return done;
}

int main() {
  std::mt19937_64 rng(31);
  const long n[] = {run<2, 1>(rng, 1500), run<2, 2>(rng, 1500), run<3, 1>(rng, 1500), run<3, 2>(rng, 3000),
                    run<3, 3>(rng, 1500)};
  long all = 0;
  for (long k : n) {
    if (k < 0) return 1;
    all += k;
  }
  std::printf("ok %ld\n", all);
  return 0;
}
