// The certified draws' bounds (lda_internal.h: kEps, draw_tau, s_bound,
// q_bound, q_bound_f) on the CPU: the sampler's single-precision arithmetic
// step by step (runs of 8 fused multiply-adds, fp64 over the runs, the walk in
// a run, the walk in a block of Q'), on rows and uniforms chosen so that x
// falls next to an edge and the roundings pull one way.  A draw that the
// bounds let stand has to be the one of 80-bit arithmetic; with the bounds cut
// to a sixteenth of what they are some are not.  Exit status 0 = every check
// held.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "lda_internal.h"

using lda::kEps;
using lda::kWScale;

namespace {
constexpr int kRunLen = 8;
typedef long double L;

struct Tally {
  long decided[3] = {0, 0, 0}, undecided[3] = {0, 0, 0}, wrong[3] = {0, 0, 0};  // by branch: M, S', Q'
  double worst_run = 0.0;  // largest error of S' seen, in units of 2^-24 of it
};

struct Token {
  std::vector<uint32_t> topic, count;  // the row, K1's entry among them
  std::vector<double> w;               // W^' of every topic (K1: 0)
  double a1, alpha, qp;
  uint32_t K1, c1;
};

// W^ just above or below a tie of its rounding to single precision, so that the error is the largest there is, or any.
double near_tie(std::mt19937_64 &g, double size, int way) {
  std::uniform_real_distribution<double> u(0.0, 1.0);
  const double any = size * (0.5 + u(g));
  if (way == 0) return any;
  const float f = float(std::ldexp(1.0 + 0x1p-3 * u(g), std::ilogb(any)));
  return double(f) * (1.0 + (way > 0 ? 1.0 : -1.0) * 0.99 * 0x1p-24);
}

void one(std::mt19937_64 &g, int bs, double scale, Tally &t) {
  std::uniform_real_distribution<double> u01(0.0, 1.0);
  const int K = 64 + int(g() % 300), way = int(g() % 3) - 1;
  const bool mix = g() % 2;
  Token k;
  k.alpha = std::ldexp(0.5 + u01(g), int(g() % 12) - 8);
  k.K1 = uint32_t(g() % uint64_t(K));
  k.w.resize(size_t(K));
  const double base = std::ldexp(0.5 + u01(g), -int(g() % 30));
  for (double &w : k.w) w = near_tie(g, base * std::ldexp(1.0, -int(g() % 8)), way);
  k.a1 = base * std::ldexp(1.0, int(g() % 10));
  k.w[k.K1] = 0.0;
  k.c1 = 0;
  for (int q = 0; q < K; ++q)
    if (g() % 4 == 0) {
      k.topic.push_back(uint32_t(q));
      k.count.push_back(1 + uint32_t(g() % (mix ? 2047 : 65535)) % (g() % 2 ? 4 : 65535));
      if (uint32_t(q) == k.K1) k.c1 = k.count.back();
    }
  const size_t n = k.topic.size(), blocks = size_t((K + bs - 1) / bs);
  if (n == 0) return;
  std::vector<float> wf(blocks * size_t(bs), 0.0f);
  std::vector<double> qb(blocks + 1, 0.0);
  L q_exact = 0;
  for (int q = 0; q < K; ++q) wf[size_t(q)] = float(k.w[size_t(q)] * kWScale);
  for (size_t b = 0; b < blocks; ++b) {
    double s = 0.0;
    for (int q = int(b) * bs; q < std::min(K, int(b + 1) * bs); ++q) s += k.alpha * k.w[size_t(q)];
    qb[b + 1] = qb[b] + s;
  }
  for (double w : k.w) q_exact += L(k.alpha) * w;
  k.qp = double(q_exact);
  // S' by runs in single precision, and exactly
  std::vector<double> run;
  L S_exact = 0;
  for (size_t r = 0; r < n; r += kRunLen) {
    float s = 0.0f;
    for (size_t q = r; q < std::min(n, r + kRunLen); ++q) {
      S_exact += L(k.count[q]) * k.w[k.topic[q]];
      s = mix ? std::fmaf(float(k.count[q]) * 0x1p-24f, wf[k.topic[q]], s) : std::fmaf(float(k.count[q]), wf[k.topic[q]], s);
    }
    run.push_back(mix ? double(s) : double(s) * (1.0 / kWScale));
  }
  double S = 0.0;
  for (double s : run) S += s;
  if (S_exact > 0) t.worst_run = std::max(t.worst_run, double(std::fabs((L(S) - S_exact) / S_exact)) * 0x1p24);
  const double M = k.a1 * (double(k.c1) + k.alpha);
  const L M_exact = L(k.a1) * (L(k.c1) + k.alpha), Z_exact = M_exact + S_exact + q_exact;

  // u next to an edge of the exact draw
  L edge = M_exact;
  const int which = int(g() % 3);
  if (which == 1) {
    const size_t to = g() % n;
    for (size_t q = 0; q <= to; ++q) edge += L(k.count[q]) * k.w[k.topic[q]];
  } else if (which == 2) {
    const size_t to = g() % uint64_t(K);
    edge += S_exact;
    for (size_t q = 0; q <= to; ++q) edge += L(k.alpha) * k.w[q];
  }
  const L off = L(u01(g) - 0.5) * std::ldexp(1.0L, -(6 + int(g() % 24)));
  const L u_l = std::floor((edge / Z_exact) * (1 + off) * 0x1p53L) * 0x1p-53L;
  if (!(u_l >= 0 && u_l < 1)) return;
  const double u = double(u_l);

  // the exact draw
  const L xe = L(u) * Z_exact;
  int branch = 0;
  uint32_t want = k.K1;
  if (!(xe < M_exact)) {
    L at = M_exact;
    bool found = false;
    for (size_t q = 0; q < n && !found; ++q) {
      at += L(k.count[q]) * k.w[k.topic[q]];
      if (xe < at) {
        want = k.topic[q];
        branch = 1;
        found = true;
      }
    }
    for (int q = 0; q < K && !found; ++q) {
      at += L(k.alpha) * k.w[size_t(q)];
      if (xe < at) {
        want = uint32_t(q);
        branch = 2;
        found = true;
      }
    }
    if (!found) return;
  }

  // the sampler's draw
  const double x = u * ((M + S) + k.qp);
  const double Su = double(float(S)) * (1.0 + 0x1p-20);
  const double tau = lda::draw_tau(k.a1 * (double(k.c1) + k.alpha), Su, k.qp) * scale;
  const double e2 = (lda::s_bound(Su, 0.0)) * scale + tau;
  uint32_t got = 0xFFFFFFFFu;  // undecided
  if (x < M) {
    if (M - x > e2) got = k.K1;
  } else if (x < M + S) {
    double start = M;
    size_t r = 0;
    while (r + 1 < run.size() && x >= start + run[r]) start += run[r++];
    const double xs = x - start;
    double p = 0.0, below = -1.0, above = 0.0;
    size_t ent = n;
    for (size_t q = r * kRunLen; q < std::min(n, (r + 1) * size_t(kRunLen)); ++q) {
      const double term = double(k.count[q]) * (double(wf[k.topic[q]]) * (1.0 / kWScale));
      if (p <= xs) {
        ent = q;
        below = p;
        above = p + term;
      }
      p += term;
    }
    if (xs - below > e2 && above - xs > e2 && below >= 0.0) got = k.topic[ent];
  } else {
    const double xs = x - (M + S);
    if (xs < qb[blocks] && xs >= 0.0) {
      const double eq1 = lda::q_bound(Su, k.qp, 0.0) * scale + tau;
      size_t lo = 0;
      while (lo + 1 < blocks && qb[lo + 1] <= xs) ++lo;
      const float inv = float(kWScale / k.alpha), xb = float((xs - qb[lo]) * (kWScale / k.alpha));
      float p = 0.0f, below = 0.0f;
      size_t at = 0;
      for (int q = 0; q < bs; ++q) {
        if (p <= xb) {
          at = size_t(q);
          below = p;
        }
        p += wf[lo * size_t(bs) + size_t(q)];
      }
      const float above = below + wf[lo * size_t(bs) + at];
      const float eq = lda::q_bound_f(eq1, inv, p * float(scale), xb * float(scale), bs);
      if (xb - below > eq && above - xb > eq) got = uint32_t(lo * size_t(bs) + at);
    }
  }
  if (got == 0xFFFFFFFFu) {
    ++t.undecided[branch];
  } else {
    ++t.decided[branch];
    if (got != want) ++t.wrong[branch];
  }
}
}  // namespace

int main() {
  for (int bs : {16, 32}) {
    std::mt19937_64 g(11 + bs);
    Tally full, cut;
    for (int q = 0; q < 100000; ++q) one(g, bs, 1.0, full);
    for (int q = 0; q < 100000; ++q) one(g, bs, 1.0 / 16, cut);
    for (int b = 0; b < 3; ++b) {
      std::printf("block %d branch %d: %ld decided, %ld undecided, %ld wrong; bounds / 16: %ld decided, %ld wrong\n", bs, b,
                  full.decided[b], full.undecided[b], full.wrong[b], cut.decided[b], cut.wrong[b]);
      if (full.wrong[b] != 0 || full.decided[b] < 1000 || full.undecided[b] < 1000 || cut.wrong[b] == 0) return 1;
    }
    std::printf("largest error of S': %.2f of 2^-24 (the bound: %.2f)\n", full.worst_run, kEps * 0x1p24);
    if (full.worst_run > kEps * 0x1p24) return 1;
  }
  std::printf("certified draw checks passed\n");
  return 0;
}
