// Where the tiles of swap_cooc_kernel lie in its dynamic LDS, and which of them a wave multiplies.  Plain arithmetic of
// host and device, apart from the kernel so that a host test can walk every shape.
#pragma once

namespace hm {

constexpr int kCoocWaves = 16;      // of a workgroup
constexpr int kCoocPartMaxE = 256;  // experts up to which the workspace holds partial tables

// Tile columns of a panel of C.
constexpr int cooc_columns(int E) { return E > 128 && E <= kCoocPartMaxE ? 2 : 1; }

// Tiles of 32 rows, one behind the other: A (all experts), S (the panel's COLS tiles), M (the cut's groups, one tile or
// two). A wave w has a row of C's tiles, its A tile by all of the panel's S tiles, or, from the last wave down, a tile
// of the panel's CG, an S tile by one M tile; with more than 448 experts and one column the last waves have both.
template <int COLS>
struct CoocTiles {
  static constexpr int kColumnsOfC = COLS, kColumnsOfG = 1;   // tiles that a row tile is multiplied by
  int a, m;
  constexpr CoocTiles(int E, int ng) : a((int)(((unsigned)E + 31u) >> 5)), m((int)(((unsigned)ng + 31u) >> 5)) {}
  constexpr int s_at() const { return 32 * a; }   // first rows
  constexpr int m_at() const { return s_at() + 32 * COLS; }
  constexpr int rows() const { return m_at() + 32 * m; }
  constexpr int g_row(int w) const { return (kCoocWaves - 1 - w) >> (m - 1); }   // of CG's tiles
  constexpr int g_column(int w) const { return (kCoocWaves - 1 - w) & (m - 1); }
  constexpr bool has_c(int w) const { return w < a; }
  constexpr bool has_g(int w) const { return g_row(w) < COLS; }
  // First rows of the row tile and of the first column tile of a product.
  constexpr int c_rows(int w) const { return 32 * w; }
  constexpr int c_columns(int) const { return s_at(); }
  constexpr int g_rows(int w) const { return s_at() + 32 * g_row(w); }
  constexpr int g_columns(int w) const { return m_at() + 32 * g_column(w); }
};

}  // namespace hm
