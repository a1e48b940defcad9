// Checks the row copy engine's map from pieces to rows and bytes (copy_geom.hpp)
// on the host, for every row width libgg accepts (4 .. 32768 bytes, multiples of
// 4), with the code the kernels run: over a tile of 64 rows, piece c must decode
// to row c / pieces, and the pieces of a row must lie inside it, at multiples of
// 4, and cover its bytes without a gap.  Prints the number of widths checked and
// exits non-zero on the first mismatch.
#include <stdint.h>
#include <stdio.h>

#include "copy_geom.hpp"

int main() {
  int widths = 0;
  for (int rb = 4; rb <= 32768; rb += 4) {
    const gg::CopyGeom g = gg::copy_geom(rb);
    const int vb = gg::copy_by_16(rb) ? 16 : 4;
    if (vb > rb || g.pieces == 0) {
      printf("row_bytes %d: pieces of %d bytes\n", rb, vb);
      return 1;
    }
    uint32_t c = 0;
    for (uint32_t row = 0; row < 64; ++row) {
      uint32_t covered = 0;              // bytes of the row from its first on
      for (uint32_t p = 0; p < g.pieces; ++p, ++c) {
        uint32_t r = ~0u;
        const uint32_t off = gg::piece_at(g, c, vb, &r);
        if (r != row || off % 4 != 0 || off > covered || off + vb > (uint32_t)rb) {
          printf("row_bytes %d vb %d: piece %u -> row %u byte %u, want row %u, a byte up to %u\n",
                 rb, vb, c, r, off, row, covered);
          return 1;
        }
        covered = off + vb;
      }
      if (covered != (uint32_t)rb) {
        printf("row_bytes %d vb %d: %u bytes covered\n", rb, vb, covered);
        return 1;
      }
    }
    ++widths;
  }
  printf("%d\n", widths);
  return 0;
}
