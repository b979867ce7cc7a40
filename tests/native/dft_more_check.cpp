// Host check of the register DFTs used as factors of the lengths in
// csrc/lengths_more.def against the O(N^2) definition in double: prints
// "N max_err_fwd max_err_inv" (errors scaled by 1/sqrt(N)).
#include <cmath>
#include <complex>
#include <cstdio>

#include "../../paper_2003_07504_amd/csrc/fft_reg.hpp"

using ilsk::cf;

template <int N, int DIR>
double check() {
  cf x[N];
  std::complex<double> in[N];
  for (int i = 0; i < N; ++i) {
    in[i] = {std::cos(0.9 * i + 0.1), std::sin(0.4 * i * i + 0.3)};
    x[i] = {(float)in[i].real(), (float)in[i].imag()};
  }
  ilsk::dft<N, DIR>(x);
  double e = 0.0;
  for (int k = 0; k < N; ++k) {
    std::complex<double> ref = 0.0;
    for (int n = 0; n < N; ++n) ref += in[n] * std::polar(1.0, DIR * 2.0 * M_PI * double((long long)n * k % N) / N);
    e = std::fmax(e, std::abs(std::complex<double>(x[k].x, x[k].y) - ref));
  }
  return e / std::sqrt((double)N);
}

template <int... Ns>
void run() {
  ((std::printf("%d %.3e %.3e\n", Ns, check<Ns, -1>(), check<Ns, 1>())), ...);
}

int main() {
  run<1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72, 75>();
  return 0;
}
