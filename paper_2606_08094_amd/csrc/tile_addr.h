// Addresses of the kernels' buffer loads from tiled operands (1 KB tiles of 16
// rows by one 64-byte k-step).  A load has an offset per lane and one that is
// uniform over the wave.  Only the lane offset is sure to be checked against
// the buffer's end, so whatever is not there (a step past the range, a subtile
// past the last row) goes past the end in the lane offset, with a uniform
// offset of 0; everything else lies inside with both offsets added.
// No includes: also compiled for the host, where the test goes through every
// lane of every shape.
#pragma once

constexpr unsigned kOob = 0x7ffffff0u;   // past the end of every buffer (they are below 2 GiB)

struct TileLoad { unsigned lane, uni; };

// Skinny GEMM, W: the workgroup's buffer holds `subs` row blocks of wt k-tiles.
// Subtile s, k-step k of the range that ends at ke; lo: the lane's place in a tile.
constexpr TileLoad skinny_w_at(unsigned lo, int s, int subs, unsigned k, unsigned ke, int wt) {
  return s < subs && k < ke ? TileLoad{lo, ((unsigned)(s * wt) + k) * 1024u} : TileLoad{kOob, 0u};
}
// Skinny GEMM, X: the buffer is the whole operand, [k-tiles][xt rows][64 bytes].
constexpr TileLoad skinny_x_at(unsigned lo, int row, int xt, unsigned k, unsigned ke) {
  return k < ke && row < xt ? TileLoad{lo, (k * (unsigned)xt + (unsigned)row) * 64u} : TileLoad{kOob, 0u};
}

// Persistent kernel's team GEMMs: k-step v of the 128 k-values at kc.  TAIL:
// K may end inside those or before them; else they all exist.
// W tiled [rows / 16][K / 32][16][32] bf16, the 16-row block that begins at `row`.
template <bool TAIL>
constexpr TileLoad team_w_at(unsigned lo, int row, int kc, int v, int K) {
  return TAIL && kc + 32 * v >= K ? TileLoad{kOob, 0u}
                                  : TileLoad{lo + 1024u * (unsigned)v,
                                             ((unsigned)(row >> 4) * (unsigned)(K >> 5) + (unsigned)(kc >> 5)) * 1024u};
}
// X [K / 32][M][32] bf16, 16-row subtile ms; lo: the lane's place in a tile, kOob in rows past M.
template <bool TAIL>
constexpr TileLoad team_x_at(unsigned lo, int ms, int kc, int v, int K, int M) {
  return TAIL && kc + 32 * v >= K ? TileLoad{kOob, 0u}
                                  : TileLoad{lo, (unsigned)(((kc >> 5) + v) * M * 64 + ms * 16 * 64)};
}
