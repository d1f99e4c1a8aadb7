// pipe_check.cpp's replay for the narrow tiles of the fp32 expert GEMMs (CG = 2), and the
// closed form of the wait counts (Pending) against pending_ok for every tile shape.
#define main wide_tiles_main
#include "pipe_check.cpp"
#undef main

template <int MB, int CG> static bool closed_form() {
  using P = ace::Pipe<MB, CG, 2, 8>;
  for (int nk = 1; nk <= 128; ++nk)
    for (int na = 0; na <= P::NA_MAX; ++na)
      for (int kt = 0; kt < nk; ++kt) {
        const int want = ace::pending_ok<P>(kt, nk, na), got = ace::Pending<P>::count(kt, nk, na);
        if (got != want || got > ace::Pending<P>::MAX) {
          std::printf("MB=%d CG=%d nk=%d na=%d kt=%d: closed form %d, count %d\n", MB, CG, nk, na, kt, got, want);
          return false;
        }
      }
  return true;
}

int main() {
  constexpr int W = 8;
  const bool ok = check<4, 2, 2, W>() && closed_form<4, 2>() &&
                  closed_form<4, 4>() && closed_form<8, 4>() && closed_form<12, 4>() && closed_form<16, 4>() &&
                  closed_form<4, 8>() && closed_form<8, 8>() && closed_form<12, 8>() && closed_form<16, 8>();
  std::printf(ok ? "ok\n" : "FAILED\n");
  return ok ? 0 : 1;
}
