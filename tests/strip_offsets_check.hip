// Host-side check of the strip tiles' load offsets (tests/test_strip_offsets.py):
// a lane keeps its offset from the operand's base in 32 bits, so no offset may
// reach 2^32 bytes at any size that a step accepts, and each must name the element
// that the tile's column stands for.  Runs without a GPU.
#include <stdio.h>

#include "rif_internal.hpp"
#include "strip64.hpp"

using namespace rif;

static long n_check = 0, n_fail = 0;
static void expect(bool ok, const char* what, long nb, long mu0, long nu0, long got) {
  ++n_check;
  if (ok) return;
  if (++n_fail <= 10) printf("FAIL %s: n_bf %ld, block (%ld, %ld), offset %ld\n", what, nb, mu0, nu0, got);
}

// Every load of the block of (mu, nu) at (mu0, nu0), one row per k apart ld.
template <class L>
static void block(const char* what, int nb, int mu0, int nu0, long ld, int nrow) {
  auto column = [&](int x) { return block_offset(x, mu0, nu0, nb); };
  for (int u = 0; u < L::NI; ++u)
    for (int lane = 0; lane < 64; ++lane) {
      const long o = strip_offset<L>(u, lane, 0, [](int) { return 0l; }, ld, column);
      expect(o >= 0 && o < (1l << 32), what, nb, mu0, nu0, o);
    }
  for (int x = 0; x < 16 * nrow; x += 2) {
    const int mu = mu0 + x / 16, p = nu0 + x % 16;
    if (mu < nb && p < nb) expect(block_offset(x, mu0, nu0, nb) + (long)mu0 * nb == (long)mu * nb + pair_start(p, nb), what, nb, mu0, nu0, x);
  }
}
template <class Cfg>
static void step(const char* what, int nb, bool slab_rows) {
  constexpr int TMU = Cfg::BN / 16;
  const long ld = slab_rows ? (long)nb * nb : 0;
  const int lm = (nb - 1) / TMU * TMU, ln = (pair_len(nb) - 1) / 16 * 16;
  for (int mu0 : {0, lm / 2 / TMU * TMU, lm - TMU, lm})
    for (int nu0 : {0, ln / 2 / 16 * 16, ln - 16, ln})
      if (mu0 >= 0 && nu0 >= 0) {
        block<Strip<Cfg, 8>>(what, nb, mu0, nu0, ld, TMU);
        block<Strip<Cfg, 1>>(what, nb, mu0, nu0, ld, TMU);
      }
}

int main() {
  int top = 0;   // the largest n_bf that the build's strips take
  for (int nb = 2; nb < 40000; ++nb)
    if (strip_fits(nb, nb, 2)) top = nb;
  expect(top > 0, "strip_fits", top, 0, 0, 0);
  for (int nb : {2, 3, 15, 16, 17, 33, 348, 5792, 5793, 5850, top - 1, top}) {
    step<StripCfg<128, 8>>("J^q, Fock", nb, true);
    step<StripCfg<64, 4>>("J^q, 64 columns", nb, true);
  }
  // the preparation's solve: one slab in the base of each load, n_bf^2 up to 2^30
  for (int nb : {2, 3, 16, 17, 23170, 23171, 32767, 32768}) step<StripCfg<128, 8>>("solve", nb, false);
  printf("%ld checks, %ld failures\n", n_check, n_fail);
  return n_fail != 0;
}
