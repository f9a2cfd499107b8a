// FP64 products of 3x3 matrices read from the library's tile-major arrays ([n][9][V] double2),
// and steps between sites: pieces of the link derivative.
#pragma once

#include "wc_kernels.h"

namespace wc {

typedef cplx<double> zc;
typedef SU3<double> Mat;

WC_D void mz(Mat& a) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) a.m[i][j] = {0.0, 0.0};
}
// c = a b
WC_D void mmul(const Mat& a, const Mat& b, Mat& c) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      zc t = a.m[i][0] * b.m[0][j];
      cmac(t, a.m[i][1], b.m[1][j]);
      cmac(t, a.m[i][2], b.m[2][j]);
      c.m[i][j] = t;
    }
}
// c += sg a b over row k of b
template <int SG> WC_D void mrow(const Mat& a, const zc* b, int k, Mat& c) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) cmac(c.m[i][j], SG > 0 ? a.m[i][k] : -a.m[i][k], b[j]);
}

// a site by its tile and its coordinates in the tile
struct Pos {
  int tc[4], lc[4], tile, s;
};
WC_D void pos_of(const Geom& g, int s, Pos& p) {
  p.s = s;
  p.tile = s / g.bvol;
  tile_coords(g, p.tile, p.tc);
  local_coords(g, s - p.tile * g.bvol, p.lc);
}
template <int MU, int DIR> WC_D Pos step(const Geom& g, const Pos& p) {
  Pos q = p;
  int ph;
  bool same;
  q.s = neighbour(g, p.s, p.tile, p.tc, p.lc, MU, DIR, &ph, &same);
  if (DIR > 0) {
    const bool over = p.lc[MU] + 1 == g.B[MU];
    q.lc[MU] = over ? 0 : p.lc[MU] + 1;
    if (over) q.tc[MU] = p.tc[MU] + 1 == g.NB[MU] ? 0 : p.tc[MU] + 1;
  } else {
    const bool over = p.lc[MU] == 0;
    q.lc[MU] = over ? g.B[MU] - 1 : p.lc[MU] - 1;
    if (over) q.tc[MU] = p.tc[MU] == 0 ? g.NB[MU] - 1 : p.tc[MU] - 1;
  }
  q.tile = ((q.tc[0] * g.NB[1] + q.tc[1]) * g.NB[2] + q.tc[2]) * g.NB[3] + q.tc[3];
  return q;
}
WC_D int lex_of(const Geom& g, const Pos& p) { return lex_index(g, p.tc, p.lc); }

// matrix n (links: direction; Xi: plane) at a site of a [n][9][V] array, or its adjoint
template <bool DAG> WC_D void mload(const double2* f, int V, int n, int s, Mat& a) {
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 v = gld_d2(f, (size_t)(n * 9 + k) * V + s);
    if (DAG)
      a.m[k % 3][k / 3] = {v.x, -v.y};
    else
      a.m[k / 3][k % 3] = {v.x, v.y};
  }
}
// row k of it alone: a product's right operand is read row by row as the product runs, so that
// it never occupies registers as a whole
template <bool DAG> WC_D void mload_row(const double2* f, int V, int n, int s, int k, zc* b) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double2 v = gld_d2(f, (size_t)(n * 9 + (DAG ? 3 * j + k : 3 * k + j)) * V + s);
    b[j] = {v.x, DAG ? -v.y : v.y};
  }
}

// planes (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
constexpr int plane_of(int a, int b) {
  const int r = a < b ? a : b, s = a < b ? b : a;
  return r == 0 ? s - 1 : r == 1 ? s + 1 : 5;
}

}  // namespace wc
