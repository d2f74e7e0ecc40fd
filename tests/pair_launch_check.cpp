// CPU driver for the launch shapes of the kernels that cover several columns a
// wave with a halo (pair_launch and density_launch of host_layout.h), built
// with the host sanitizers by tests/test_pair_launch.py.  The kernels divide
// the grid themselves, from nstrips and rows; this forms their division and
// checks that every site has exactly one owner, that no wave owns more columns
// than it holds, that the blocks hold every wave and that the diagnostic
// partials and the state's byte offsets fit.  Prints "ok <cases>".
#include <cstdio>
#include <cstdlib>

#include "host_layout.h"

using namespace lbe;
using namespace lbe::host;

static bool check(const PairLaunch &L, const lbe_csf_params &p, size_t bytes, int cols) {
  const int nx = p.nx, ny = p.ny;
  if (L.nblocks == 0) return L.rows == 0 && L.nparts == 0;   // not taken
  if (ny < 8 || bytes > kPairMaxBytes || L.nstrips < 1 || L.rows < 1) return false;
  const int wx = (nx + L.nstrips - 1) / L.nstrips;
  if (wx > cols || (long)L.nstrips * wx < nx || (long)(L.nstrips - 1) * wx >= nx) return false;
  const int nchunks = (ny + L.rows - 1) / L.rows;
  if ((long)(nchunks - 1) * L.rows >= ny) return false;
  if (L.nparts != L.nstrips * nchunks) return false;
  if (L.tile) return L.tile == L.rows && L.nblocks == L.nparts && (L.tile == 2 || L.tile == 4 ||
                     (L.tile == 8 && p.precision == LBE_CSF_FP32_DEV));
  const int most = p.precision == LBE_CSF_FP32_DEV ? 8 : 4;
  return L.nw >= 1 && L.nw <= most && L.nblocks == (L.nstrips + L.nw - 1) / L.nw * nchunks;
}

int main() {
  long cases = 0;
  const int nys[] = {3, 7, 8, 9, 15, 17, 64, 100, 255, 513, 777, 1024, 2049, 4096, 9001};
  for (const char *over : {"", "0", "1", "2"}) {
    if (*over) setenv("LBE_CSF_PAIR", over, 1);
    for (const char *rows : {"", "1", "3", "4", "8", "100000"}) {
      if (*rows) setenv("LBE_CSF_PAIR_ROWS", rows, 1);
      else unsetenv("LBE_CSF_PAIR_ROWS");
      for (int nx = 3; nx < 9000; nx += nx < 700 ? 1 : 97)
        for (int ny : nys)
          for (int prec : {LBE_CSF_FP32_DEV, LBE_CSF_FP64})
            for (double rho2 : {0.0, 0.5}) {
              lbe_csf_params p{};
              p.nx = nx, p.ny = ny, p.walls_y = 1, p.precision = prec;
              p.rho = 1.0, p.rho2 = rho2;
              const size_t n = (size_t)nx * ny;
              const size_t bytes = prec == LBE_CSF_FP64 ? state_bytes_for<double>(n)
                                                        : state_bytes_for<float>(n);
              const bool two = two_densities(&p);
              const PairLaunch L = two ? density_launch(&p, bytes) : pair_launch(&p, bytes);
              if (!check(L, p, bytes, two ? 64 - 2 * kDensityHalo : kPairCols)) {
                std::fprintf(stderr, "FAIL %d x %d prec %d rho2 %g pair '%s' rows '%s': nw %d "
                             "nstrips %d rows %d nblocks %d nparts %d tile %d\n", nx, ny, prec,
                             rho2, over, rows, L.nw, L.nstrips, L.rows, L.nblocks, L.nparts,
                             L.tile);
                return 1;
              }
              ++cases;
            }
    }
  }
  std::printf("ok %ld\n", cases);
  return 0;
}
