// Geometry of the row copy engine: how a row is cut into pieces of 16 bytes (4
// for rows below 16 bytes) and how a piece's index within a tile of rows maps
// back to its row and byte.  Plain integer code, shared by the host (which
// fills the struct) and the kernels (which decode piece indices); it needs no
// HIP header, so that a host program can check the map for every row width the
// library accepts.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define GG_HD __host__ __device__
#else
#define GG_HD
#endif

namespace gg {

// Rows of 16 bytes and more move in 16-byte pieces whatever their alignment
// (every base and stride is a multiple of 4, which is all the hardware's
// 16-byte accesses need); narrower rows in words.
inline bool copy_by_16(int32_t row_bytes) { return row_bytes >= 16; }

// A row is `pieces` pieces of VB bytes, piece p at byte min(p * VB, last).  A row
// that is not a multiple of 16 bytes ends in a piece that overlaps the one
// before (both write the same bytes there), so that its last words need no pass
// of their own.
struct CopyGeom {
  uint32_t pieces;
  uint32_t pmagic;    // div_magic(pieces)
  uint32_t last;      // row_bytes - VB
};

// Multiplier for c / d as the high word of c * magic: magic = ceil(2^32 / d).
// With e = magic * d - 2^32 (0 <= e < d) the quotient is exact while
// c * e < 2^32; a tile has at most 64 rows, so c < 64 d and d <= 8192
// suffices (d is at most 32768 / 16 for rows).  A divisor of 1 has no 32-bit
// multiplier (2^32 does not fit), so it is marked by magic = 0 and
// chunk_row returns c itself.
GG_HD inline uint32_t div_magic(uint32_t d) {
  return d > 1 ? (uint32_t)(((1ULL << 32) + d - 1) / d) : 0u;
}

// Row of chunk c, for a divisor whose multiplier is `magic`.
GG_HD inline uint32_t chunk_row(uint32_t c, uint32_t magic) {
  return magic ? (uint32_t)(((uint64_t)c * magic) >> 32) : c;
}

// Row and byte of piece c of a tile.
GG_HD inline uint32_t piece_at(const CopyGeom& g, uint32_t c, int vb, uint32_t* row) {
  const uint32_t r = chunk_row(c, g.pmagic);
  const uint32_t off = (c - r * g.pieces) * (uint32_t)vb;
  *row = r;
  return off < g.last ? off : g.last;
}

inline CopyGeom copy_geom(int32_t row_bytes) {
  const int vb = copy_by_16(row_bytes) ? 16 : 4;
  CopyGeom g;
  g.pieces = (uint32_t)((row_bytes + vb - 1) / vb);
  g.pmagic = div_magic(g.pieces);
  g.last = (uint32_t)(row_bytes - vb);
  return g;
}

}  // namespace gg
