// Host check of the pieces of j-splits (piece_range, piece_follows) over every
// tile count, split length and piece length up to a bound: the pieces cover
// every tile once, in order, and a piece reads the minima of exactly the
// earlier tiles of its split, all of which the first launch computes; an empty
// piece reads none.  Prints one line per violated case and the number of
// cases; exits 1 on any violation.  Built and run by
// tests/test_pieces_host.py; it calls no HIP runtime function.
#include "../../paper_0902_4463_amd/csrc/g6mi_device.h"

#include <cstdio>

using namespace g6mi;

int main() {
  long cases = 0, bad = 0;
  for (int ntiles = 1; ntiles <= 70; ++ntiles)
    for (int vper = 1; vper <= ntiles; ++vper)
      for (int per = 1; per <= vper; ++per) {
        PieceArgs pc;
        pc.vper = vper;
        pc.per = per;
        const int npieces = (ntiles + vper - 1) / vper * ((vper + per - 1) / per);
        int next = 0; // the first tile no piece has had
        bool ok = true;
        for (int y = 0; y < npieces; ++y) {
          const PieceRange r = piece_range(pc, ntiles, y);
          for (int tt = r.split; tt < r.begin; ++tt) ok = ok && tt >= 0 && tt < ntiles && piece_follows(pc, ntiles, tt);
          if (r.begin < r.end) {
            ok = ok && r.begin == next && r.end <= ntiles && r.begin / vper * vper == r.split;
            next = r.end;
          } else {
            ok = ok && r.begin == r.split;
          }
        }
        ok = ok && next == ntiles;
        // tiles from the last split's first on are that split's
        const int vlast = (ntiles - 1) / vper * vper;
        for (int tt = 0; tt < ntiles; ++tt) ok = ok && (tt >= vlast) == (tt - tt % vper == vlast);
        ++cases;
        if (!ok && ++bad <= 20) std::printf("violated: ntiles=%d vper=%d per=%d\n", ntiles, vper, per);
      }
  std::printf("cases %ld violations %ld\n", cases, bad);
  return bad ? 1 : 0;
}
