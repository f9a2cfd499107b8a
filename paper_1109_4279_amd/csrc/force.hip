// Gauge-link derivative of Re<Y, D X> and the pseudofermion force.
//
// The solves of arXiv:1109.4279 feed the HMC force from the fermion determinant
// (Sec. 1).  For S = phi^dag (D^dag D)^-1 phi, Y = D^-dag phi and X = D^-1 Y,
// dS = -2 Re<Y, dD X>.  This file computes, per link, the matrix K_mu(x) with
//   d Re<Y, D X> = Re tr(dU_mu(x) K_mu(x))        for any complex dU,
// from two parts:
//   hopping: K += -1/2 ph sum_t [ X(x+mu)_t ((1-g_mu) Y(x))_t^dag + ((1+g_mu) Y(x+mu))_t X(x)_t^dag ]
//   clover : with Xi_{rs}(y) = (i c_sw/16)(G + G^dag), G_{rs}(y) = sum_{st} (sigma_rs)_{st} X_t(y) Y_s(y)^dag,
//            every plaquette leaf W1 W2 W3 W4 at y that contains the link at position i adds
//            W_{i+1}..W_4 Xi(y) W_1..W_{i-1} (or its dagger when the leaf runs the link backwards).
//
// A link lies in two plaquettes of each plane that contains it; with a, b, c the other three
// factors of one in order (a staple) and Xi at its corners, the four leaves that are this
// plaquette add
//   Xi(x+mu) abc + a Xi b c + a b Xi c + abc Xi(x),
// and, Xi being anti-Hermitian, a plaquette that runs the link backwards adds the same with
// the opposite sign.  So per plane, with S_up, S_down the staples abc and eps = +1 for
// mu < nu, -1 otherwise,
//   K += eps [ Xi(x+mu) (S_up - S_down) + (S_up - S_down) Xi(x) + T_up - T_down ],
//   T = ((a Xi_2) b + (a b) Xi_3) c,
// 14 products of 3x3 matrices and 12 matrices read per plane (24 and 40 leaf by leaf).
//
// The links and Xi are read in the tile-major structure-of-arrays storage; a link's three
// planes and its hopping part are four wavefronts' work, a gather, so that no two lanes write
// the same output.  Bound by the matrices' trips from L2 (36 of 144 bytes a link).  Leaf by
// leaf from the canonical array (144-byte strides between lanes) the link kernel took 610 us
// at 16^3 x 32 and 274 us at 12^3 x 24, now 278 and 102 us; Xi 88 -> 38 us (its bytes take
// 34 us at the rate of a device copy).
#include "wc_su3.h"

namespace wc {

WC_D void spin(const double2* F, int V, int r, int x, zc (*v)[3]) {
  const double2* p = F + ((size_t)r * V + x) * 12;
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const double2 z = gld_d2(p, k);
    v[k / 3][k % 3] = {z.x, z.y};
  }
}

// pass 1: Xi_{rs}(y) for the six planes, summed over right-hand sides.  In the chiral basis
// sigma_{0l} = diag(sigma_l, -sigma_l) and sigma_{jk} = -eps_{jkl} diag(sigma_l, sigma_l), so
// the planes (0,l) and (j,k) come from S^c_l = sum_st (sigma_l)_st X_t Y_s^dag of the two
// chiralities c.  l = 1, 2 share their two outer products; a second pass over the spinors
// takes l = 3 (all six S^c_l at once would not fit the registers).
__global__ __launch_bounds__(WG) void k_force_xi(Geom g, const double2* Y, const double2* X, int nrhs, double csw,
                                                 double2* xi) {
  const int s = blockIdx.x * WG + threadIdx.x;
  if (s >= g.V) return;
  Pos pos;
  pos_of(g, s, pos);
  const int x0 = lex_of(g, pos);
  const double f = csw / 16.0;
  // i f (G + G^dag) for G = u S^+ + v S^-
  auto put = [&](int p, const Mat* S, double u, double v) {
    Mat G;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) G.m[a][b] = u * S[0].m[a][b] + v * S[1].m[a][b];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const zc h = f * timesI(G.m[a][b] + conj(G.m[b][a]));
        xi[(size_t)(p * 9 + a * 3 + b) * g.V + s] = make_double2(h.re, h.im);
      }
  };
  auto outer = [&](Mat& M, const zc* x, const zc* y) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) cmac_conj(M.m[a][b], y[b], x[a]);
  };
  {
    Mat A[2], B[2];  // X_1 Y_0^dag and X_0 Y_1^dag of either chirality
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      mz(A[c]);
      mz(B[c]);
    }
    for (int r = 0; r < nrhs; ++r) {
      zc x[4][3], y[4][3];
      spin(X, g.V, r, x0, x);
      spin(Y, g.V, r, x0, y);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        outer(A[c], x[2 * c + 1], y[2 * c]);
        outer(B[c], x[2 * c], y[2 * c + 1]);
      }
    }
    Mat S[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) S[c].m[a][b] = A[c].m[a][b] + B[c].m[a][b];
    put(plane_of(0, 1), S, 1.0, -1.0);
    put(plane_of(2, 3), S, -1.0, -1.0);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) S[c].m[a][b] = timesI(B[c].m[a][b] - A[c].m[a][b]);
    put(plane_of(0, 2), S, 1.0, -1.0);
    put(plane_of(1, 3), S, 1.0, 1.0);  // eps_{132} = -1
  }
  {
    Mat S[2];
    mz(S[0]);
    mz(S[1]);
    for (int r = 0; r < nrhs; ++r) {
      zc x[4][3], y[4][3];
      spin(X, g.V, r, x0, x);
      spin(Y, g.V, r, x0, y);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        outer(S[c], x[2 * c], y[2 * c]);
        const zc n[3] = {-x[2 * c + 1][0], -x[2 * c + 1][1], -x[2 * c + 1][2]};
        outer(S[c], n, y[2 * c + 1]);
      }
    }
    put(plane_of(0, 3), S, 1.0, -1.0);
    put(plane_of(1, 2), S, -1.0, -1.0);
  }
}

// hopping part of K_MU(x):  -1/2 ph sum_t [ X(x+mu)_t ((1-g_mu) Y(x))_t^dag
//                                           + ((1+g_mu) Y(x+mu))_t X(x)_t^dag ]
// (1 -+ g_mu) has rank two: its lower spins are a phase times its upper ones, so both sums run
// over two spins of projected half spinors.
template <int MU>
WC_D void force_hop(const double2* Y, const double2* X, int V, int nrhs, int x0, int xp, double ph, Mat& K) {
  for (int r = 0; r < nrhs; ++r) {
    Spinor<double> Xs, Xp, Ys, Yp;
    spin(X, V, r, x0, Xs.c);
    spin(X, V, r, xp, Xp.c);
    spin(Y, V, r, x0, Ys.c);
    spin(Y, V, r, xp, Yp.c);
    // (1 - g) is Hermitian and (1 - g)^2 = 2 (1 - g), and w^dag (1 - g) v is the product of the
    // two projected upper halves: sum_t a_t ((1 - g) b)_t^dag = P(a) P(b)^dag
    const Half<double> xm = project<double, MU, -1>(Xp), ym = project<double, MU, -1>(Ys);
    const Half<double> yp = project<double, MU, +1>(Yp), xs = project<double, MU, +1>(Xs);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        zc acc = {0.0, 0.0};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          cmac_conj(acc, ym.c[t][b], xm.c[t][a]);
          cmac_conj(acc, xs.c[t][b], yp.c[t][a]);
        }
        K.m[a][b] = K.m[a][b] + (-0.5 * ph) * acc;
      }
  }
}

// one staple of plane (MU, NU): D += eps S, K += eps T (up), or minus them (down).  The
// barriers keep the loads of later products from being hoisted over this one's registers.
template <int MU, int NU, int DIR>
WC_D void force_staple(const Geom& g, const double2* U, const double2* xi, const Pos& p, const Pos& pm, Mat& D, Mat& K) {
  constexpr int PL = plane_of(MU, NU);
  constexpr int SG = (MU < NU) == (DIR > 0) ? 1 : -1;
  const Pos pn = step<NU, DIR>(g, p);            // x +- nu
  const int smn = step<NU, DIR>(g, pm).s;        // x + mu +- nu
  Mat a, w, q, ab;
  zc b[3];
  // up: a = U_nu(x+mu), b = U_mu(x+nu)^dag, c = U_nu(x)^dag
  // down: a = U_nu(x+mu-nu)^dag, b = U_mu(x-nu)^dag, c = U_nu(x-nu)
  mload<(DIR < 0)>(U, g.V, NU, DIR > 0 ? pm.s : smn, a);
  mz(w);
#pragma unroll
  for (int k = 0; k < 3; ++k) {  // w = a Xi_2
    mload_row<false>(xi, g.V, PL, smn, k, b);
    mrow<1>(a, b, k, w);
  }
  __builtin_amdgcn_sched_barrier(0);
  mz(q);
  mz(ab);
#pragma unroll
  for (int k = 0; k < 3; ++k) {  // q = a Xi_2 b, ab = a b
    mload_row<true>(U, g.V, MU, pn.s, k, b);
    mrow<1>(w, b, k, q);
    mrow<1>(a, b, k, ab);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 3; ++k) {  // q += a b Xi_3
    mload_row<false>(xi, g.V, PL, pn.s, k, b);
    mrow<1>(ab, b, k, q);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 3; ++k) {  // T = q c, S = a b c
    mload_row<(DIR > 0)>(U, g.V, NU, DIR > 0 ? p.s : pn.s, k, b);
    mrow<SG>(q, b, k, K);
    mrow<SG>(ab, b, k, D);
  }
  __builtin_amdgcn_sched_barrier(0);
}

template <int MU, int NU>
WC_D void force_plane(const Geom& g, const double2* U, const double2* xi, const Pos& p, const Pos& pm, Mat& K) {
  constexpr int PL = plane_of(MU, NU);
  Mat D, t;
  zc b[3];
  mz(D);
  force_staple<MU, NU, +1>(g, U, xi, p, pm, D, K);
  force_staple<MU, NU, -1>(g, U, xi, p, pm, D, K);
  mload<false>(xi, g.V, PL, pm.s, t);
#pragma unroll
  for (int k = 0; k < 3; ++k) mrow<1>(t, D.m[k], k, K);  // Xi(x+mu) D
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 3; ++k) {  // D Xi(x)
    mload_row<false>(xi, g.V, PL, p.s, k, b);
    mrow<1>(D, b, k, K);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// K_MU of the work-group's 64 sites: wavefronts 0..2 take the planes, wavefront 3 the hopping
// part, and the sum goes through LDS.  (One lane with all three planes and the hopping part
// spills whatever the order; this way a path has one plane, and a quarter of the serial work.)
template <int MU>
WC_D void force_link(const Geom& g, const double2* U, const double2* Y, const double2* X, int nrhs, double csw,
                     const double2* xi, double coef, int out_kind, double2* out, int s0, double2* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s = min(s0 + lane, g.V - 1);
  Pos p;
  pos_of(g, s, p);
  Mat K;
  mz(K);
  {
    const Pos pm = step<MU, +1>(g, p);
    if (wave == 3) {
      const bool last = p.tc[0] == g.NB[0] - 1 && p.lc[0] == g.B[0] - 1;
      force_hop<MU>(Y, X, g.V, nrhs, lex_of(g, p), lex_of(g, pm), (MU == 0 && last) ? double(g.bc_t) : 1.0, K);
    } else if (csw != 0.0) {
      if (wave == 0)
        force_plane<MU, (MU + 1) & 3>(g, U, xi, p, pm, K);
      else if (wave == 1)
        force_plane<MU, (MU + 2) & 3>(g, U, xi, p, pm, K);
      else
        force_plane<MU, (MU + 3) & 3>(g, U, xi, p, pm, K);
    }
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) lds[(wave * 9 + k) * 64 + lane] = make_double2(K.m[k / 3][k % 3].re, K.m[k / 3][k % 3].im);
  __syncthreads();
  if (wave != 0 || s0 + lane >= g.V) return;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    zc t = K.m[k / 3][k % 3];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const double2 v = lds[(w * 9 + k) * 64 + lane];
      t = {t.re + v.x, t.im + v.y};
    }
    K.m[k / 3][k % 3] = t;
  }
  double2* o = out + ((size_t)MU * g.V + lex_of(g, p)) * 9;
  if (out_kind == 0) {  // torch-convention gradient G = coef * K^dag
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const zc v = coef * conj(K.m[b][a]);
        o[a * 3 + b] = make_double2(v.re, v.im);
      }
  } else {  // Lie-algebra force TA(U K) * coef
    Mat u, UK;
    mload<false>(U, g.V, MU, s, u);
    mmul(u, K, UK);
    Mat A;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) A.m[a][b] = 0.5 * (UK.m[a][b] - conj(UK.m[b][a]));
    const zc tr = A.m[0][0] + A.m[1][1] + A.m[2][2];
#pragma unroll
    for (int a = 0; a < 3; ++a) A.m[a][a] = A.m[a][a] - (1.0 / 3.0) * tr;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const zc v = coef * A.m[a][b];
        o[a * 3 + b] = make_double2(v.re, v.im);
      }
  }
}

// pass 2: K_mu(x) (hopping + clover), then the requested output; the four directions of 64
// sites are neighbouring work-groups of one XCD
__global__ __launch_bounds__(WG, 2) void k_force_link(Geom g, const double2* U, const double2* Y, const double2* X,
                                                   int nrhs, double csw, const double2* xi, double coef,
                                                   int out_kind, double2* out) {
  __shared__ double2 lds[4 * 9 * 64];
  const int it = xcd_remap(blockIdx.x, gridDim.x);
  const int s0 = (it >> 2) * 64;
  switch (it & 3) {
    case 0: force_link<0>(g, U, Y, X, nrhs, csw, xi, coef, out_kind, out, s0, lds); break;
    case 1: force_link<1>(g, U, Y, X, nrhs, csw, xi, coef, out_kind, out, s0, lds); break;
    case 2: force_link<2>(g, U, Y, X, nrhs, csw, xi, coef, out_kind, out, s0, lds); break;
    default: force_link<3>(g, U, Y, X, nrhs, csw, xi, coef, out_kind, out, s0, lds); break;
  }
}

// links64: the library's FP64 links; Y, X canonical spinors; xi_work: 54 V complex numbers
// (null when csw is 0); out canonical links
void launch_force(const Geom& g, const void* links64, const void* Y, const void* X, int nrhs, double csw, double coef,
                  int out_kind, void* xi_work, void* out, hipStream_t st) {
  const int chunks = (g.V + WG - 1) / WG;
  if (csw != 0.0)
    hipLaunchKernelGGL(k_force_xi, dim3(chunks), dim3(WG), 0, st, g, (const double2*)Y, (const double2*)X, nrhs, csw,
                       (double2*)xi_work);
  hipLaunchKernelGGL(k_force_link, dim3(4 * ((g.V + 63) / 64)), dim3(WG), 0, st, g, (const double2*)links64, (const double2*)Y,
                     (const double2*)X, nrhs, csw, (const double2*)xi_work, coef, out_kind, (double2*)out);
}

}  // namespace wc
