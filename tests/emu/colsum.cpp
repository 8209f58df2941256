// k_cg_colsum over the emulation (includes the generated cg.cpp): the launch
// that sums the F^T p partials and ends the iteration, at the last iteration
// allowed and at one where the last column has just stopped.
#include "cg.cpp"

#include <cstdio>

int main() {
  using namespace sdgp;
  constexpr int R = 3, n1 = 5, nbu = 70;
  int bad = 0;
  for (int last = 0; last < 2; ++last) {
    std::vector<double> part((size_t)n1 * R * nbu), red((size_t)n1 * R, -1.0);
    for (size_t k = 0; k < part.size(); ++k) part[k] = (double)(k % 97);
    std::vector<int32_t> act(2 * R, last ? 1 : 0);
    int32_t done = 0, it = 6;
    CgArgs A = {};
    A.R = R;
    A.n1 = n1;
    A.nbu = nbu;
    A.max_iter = last ? it + 1 : 100;
    A.p_part = part.data();
    A.p_red = red.data();
    A.st.act = act.data();
    A.st.done = &done;
    A.st.it = &it;
    ::emu::Cfg(dim3(n1 * R + 1, 1, 1), dim3(kSumT), 0, nullptr).launch("k_cg_colsum", k_cg_colsum, (const CgArgs*)&A, 2);
    for (int c = 0; c < n1 * R; ++c) {
      double s = 0.0;
      for (int b = 0; b < nbu; ++b) s += part[(size_t)c * nbu + b];
      if (red[c] != s) {
        std::printf("case %d sum %d: %g, not %g\n", last, c, red[c], s);
        ++bad;
      }
    }
    if (it != 7 || done != (last ? 0 : 7)) {
      std::printf("case %d: it %d done %d\n", last, it, done);
      ++bad;
    }
  }
  std::printf("%d wrong\n", bad);
  return bad ? 1 : 0;
}
