// Host build of the two-stage line transforms (csrc/fft_radix.h): the wide in-register
// DFTs, and every length 2..400 that two_stage splits, against a direct double-precision
// DFT.  Built with hipcc --offload-host-only by test_fft_two_stage_cpu.py; prints
//   dft R s err | two N R0 R1 s err
#include <math.h>
#include <stdio.h>

#include <random>
#include <vector>

#include "../paper_2606_01598_amd/csrc/fft_radix.h"

static double max_rel(const std::vector<float2>& x, const std::vector<float2>& got, double s) {
  const int n = int(x.size());
  double num = 0.0, den = 0.0;
  for (int k = 0; k < n; ++k) {
    double re = 0.0, im = 0.0;
    for (int t = 0; t < n; ++t) {
      const double a = s * 2.0 * M_PI * double((long(t) * k) % n) / n;
      re += x[t].x * cos(a) - x[t].y * sin(a);
      im += x[t].x * sin(a) + x[t].y * cos(a);
    }
    num = fmax(num, hypot(got[k].x - re, got[k].y - im));
    den = fmax(den, hypot(re, im));
  }
  return num / den;
}

int main() {
  std::mt19937 g(11);
  std::normal_distribution<float> nd;
  for (int R : pme::kWideRadices)
    for (float s : {-1.0f, 1.0f})
      pme::with_wide_radix(R, [&](auto rc) {
        constexpr int C = decltype(rc)::value;
        float2 v[C];
        std::vector<float2> x(C);
        for (int r = 0; r < C; ++r) x[r] = v[r] = make_float2(nd(g), nd(g));
        pme::Dft<C>::run(v, s);
        printf("dft %d %d %.3e\n", C, int(s), max_rel(x, std::vector<float2>(v, v + C), s));
      });
  for (int N = 2; N <= 400; ++N) {
    const pme::TwoStage t = pme::two_stage(N);
    if (!t.R0) continue;
    std::vector<float2> tw(N), x(N), y(N), rows(pme::two_stage_words(t.R0, t.R1));
    for (int k = 0; k < N; ++k) {
      const double a = -2.0 * M_PI * double(k) / double(N);
      tw[k] = make_float2(float(cos(a)), float(sin(a)));
    }
    for (auto& v : x) v = make_float2(nd(g), nd(g));
    for (float s : {-1.0f, 1.0f}) {
      // both orders of the radices (the x pass inverts with them in reverse)
      const int A = s < 0 ? t.R0 : t.R1, B = s < 0 ? t.R1 : t.R0;
      for (int j = 0; j < B; ++j)
        pme::with_wide_radix(A, [&](auto rc) {
          pme::two_stage_first<decltype(rc)::value>([&](int i) { return x[i]; }, rows.data(), j, B, s);
        });
      for (int j = 0; j < A; ++j)
        pme::with_wide_radix(B, [&](auto rc) {
          pme::two_stage_second<decltype(rc)::value>(
              rows.data(), [&](int i, float2 v) { y[i] = v; }, j, A, tw.data(), s);
        });
      printf("two %d %d %d %d %.3e\n", N, t.R0, t.R1, int(s), max_rel(x, y, s));
    }
  }
  return 0;
}
