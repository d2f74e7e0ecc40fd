// Placement of the moment tape in a record's region (adj_place_tape): inside
// the bytes at hand, clear of every buffer that is in use with it, and all
// steps or the last ones that fit.
#include <cstdio>
#include <cstdlib>

#include "host_layout.h"

using namespace lbe;

static void check(bool ok, const char *what, long long N, size_t avail) {
  if (ok) return;
  std::fprintf(stderr, "%s: N = %lld, %zu bytes\n", what, N, avail);
  std::exit(1);
}

int main() {
  long cases = 0, full = 0, part = 0;
  for (int nx : {3, 57, 256, 4096})
    for (int ny : {3, 100, 1024})
      for (size_t vb : {4, 8})
        for (long long N : {1LL, 2LL, 3LL, 7LL, 23LL, 100LL, 146LL, 200LL, 4000LL, 1LL << 50})
          for (int x = 0; x < 8; ++x) {
            const size_t n = (size_t)nx * ny, state = n * (vb == 8 ? 216 : 112);
            const AdjLayout B = adj_layout(nx, ny, state, vb, N);
            // avail: less than the least, the least, and more
            const size_t more[8] = {0, 0, 1, B.mom_bytes - 1, B.mom_bytes, 5 * B.mom_bytes,
                                    B.off_lam, 300 * B.mom_bytes};
            const size_t avail = x == 0 ? B.total - 1 : B.total + more[x];
            AdjLayout A = B;
            adj_place_tape(A, avail);
            if (x == 0) {
              check(A.direct == 0 && A.total == B.total, "too small a region", N, avail);
              continue;
            }
            check(A.total <= avail && A.total >= B.total, "total", N, avail);
            check(A.direct >= 0 && A.direct <= N, "steps", N, avail);
            const size_t tape = (size_t)A.direct * A.mom_bytes;
            // the cotangents and sums keep their sizes, in their order
            check(A.off_part - A.off_lam == B.off_part - B.off_lam &&
                      A.off_tw - A.off_part == B.off_tw - B.off_part &&
                      A.off_out - A.off_tw == B.off_out - B.off_tw,
                  "cotangents", N, avail);
            check((2 * 27 + 3 + kAdjA) * A.plane_bytes <= A.off_part - A.off_lam, "planes", N, avail);
            if (A.direct == N) {   // no checkpoints: the tape may take their place
              check(A.off_direct + tape <= A.off_lam || A.off_direct >= B.total, "all taped", N, avail);
              check(A.off_direct + tape <= A.total && A.off_out + 256 <= A.total, "end", N, avail);
              ++full;
            } else {
              check(A.off_lam == B.off_lam && A.off_direct == B.total && A.off_direct + tape <= avail,
                    "last steps taped", N, avail);
              check(avail - A.off_direct - tape < A.mom_bytes, "room left", N, avail);
              part += A.direct > 0;
            }
            // up to 100 steps the least region holds them all in FP32
            if (N <= 100 && N >= 7 && vb == 4) check(A.direct == N, "short runs", N, avail);
            ++cases;
          }
  std::printf("ok %ld full %ld part %ld\n", cases, full, part);
  return full && part ? 0 : 1;
}
