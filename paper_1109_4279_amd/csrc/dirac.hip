// D_w on the full lattice and its Dirichlet-block restriction, all storage precisions.
//
// The operator (Wilson-Dirac with clover term, arXiv:1109.4279 abstract and Sec. 4):
//   (D psi)(x) = A(x) psi(x) - 1/2 sum_mu [ (1 - gamma_mu) U_mu(x) psi(x+mu)
//                                          + (1 + gamma_mu) U_mu(x-mu)^dag psi(x-mu) ]
// with A(x) the two 6x6 Hermitian chiral clover blocks (which include 4 + m0).
// Block mode drops every hop whose neighbour lies in another tile (Sec. 4: the
// blocks are solved with Dirichlet boundary conditions).
//
// One lane per site, NR right-hand sides per lane: each link and clover block is
// loaded once and applied to NR spinors.  The kernel is HBM-bound; neighbour
// spinors come mostly from L2 because tiles of one XCD are spatially contiguous.
#include "wc_kernels.h"

namespace wc {

template <class R> WC_D void g5(Spinor<R>& p) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    p.c[2][a] = -p.c[2][a];
    p.c[3][a] = -p.c[3][a];
  }
}

template <class R, class T> WC_D Spinor<R> to_real(const Spinor<T>& p) {
  Spinor<R> o;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) o.c[i][c] = {R(p.c[i][c].re), R(p.c[i][c].im)};
  return o;
}

// STAGE: every work item is one 256-site tile (Schwarz blocks of 256 sites); the tile's
// input spinors are decoded once into LDS and the in-tile neighbours are read from there,
// so each spinor leaves HBM/L2 once per tile instead of once per neighbour.
// PIN: storage precision of the input (FP64 and FP32 arithmetic may read an input of
// another storage, widened or rounded to the arithmetic's precision; the 16-bit launches
// read their own precision).
template <int P, int NR, bool STAGE, int PIN = P>
__global__ __launch_bounds__(WG) void k_dirac(DiracLaunch a) {
  typedef typename Real<P>::T R;
  __shared__ double red[(WG / 64) * NR];
  extern __shared__ double stage_d[];
  cplx<R>* st_sp = (cplx<R>*)stage_d;        // [NR][12][WG] input spinors of the tile (unscaled)
  R* st_sc = (R*)(st_sp + NR * 12 * WG);     // [NR][WG] their site scales
  if (cycle_dead(a.dead)) return;
  for (int it0 = blockIdx.x; it0 < a.nitems; it0 += gridDim.x) {
    const WorkItem w = load_uniform(a.items, xcd_remap(it0, a.nitems));
    const LatDesc L = load_uniform(a.lats, w.lat);
    const Geom g = L.g;
    bool any = true;
    if (a.skip) {
      any = false;
      for (int r = 0; r < w.nr; ++r) any |= (a.skip[L.sys0 + w.rhs0 + r] == 0);
    }
    if (!any) continue;
    const int s_raw = w.chunk * WG + threadIdx.x;
    const bool valid = s_raw < g.V;
    const int s = valid ? s_raw : g.V - 1;
    const int tile = s / g.bvol;
    int tc[4], lc[4];
    tile_coords(g, tile, tc);
    local_coords(g, s - tile * g.bvol, lc);

    FieldRef fin[NR], fout[NR], fy[NR];
    const int sb = spinor_site_bytes(P), sbin = spinor_site_bytes(PIN);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int rr = w.rhs0 + (r < w.nr ? r : 0);
      const long long off = L.foff + (long long)rr * g.V;
      fin[r] = {(char*)a.in + off * sbin, a.in_sc ? (float*)a.in_sc + off : nullptr, g.V};
      fout[r] = {(char*)a.out + off * sb, a.out_sc ? a.out_sc + off : nullptr, g.V};
      fy[r] = {a.y ? (char*)a.y + off * sb : nullptr, a.y_sc ? (float*)a.y_sc + off : nullptr, g.V};
    }

    Spinor<R> acc[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) zero(acc[r]);
    if (STAGE) {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        Spinor<R> p = to_real<R>(SpinorIO<PIN>::load_raw(fin[r], s));
#pragma unroll
        for (int k = 0; k < 12; ++k) st_sp[(r * 12 + k) * WG + threadIdx.x] = p.c[k / 3][k % 3];
        st_sc[r * WG + threadIdx.x] = SpinorIO<PIN>::scale(fin[r], s);
      }
      __syncthreads();
    }
    // input spinor r at site n: from the staged tile when n is in it, else from memory
    auto in_raw = [&](int r, int n, bool in_tile, R& sc) {
      Spinor<R> p;
      if (STAGE && in_tile) {
        const int ln = n - tile * WG;
#pragma unroll
        for (int k = 0; k < 12; ++k) p.c[k / 3][k % 3] = st_sp[(r * 12 + k) * WG + ln];
        sc = st_sc[r * WG + ln];
      } else {
        p = to_real<R>(SpinorIO<PIN>::load_raw(fin[r], n));
        sc = SpinorIO<PIN>::scale(fin[r], n);
      }
      return p;
    };

    auto hop = [&](auto MUc) {
      constexpr int MU = decltype(MUc)::value;
      int ph;
      bool same;
      // forward: (1 - gamma_mu) U_mu(x) psi(x + mu)
      int nf = neighbour(g, s, tile, tc, lc, MU, +1, &ph, &same);
      // 16-bit storage: links and spinors are used unscaled and the site scales folded
      // into the one weight of the hop
      if (!a.block || same) {
        SU3<R> u = LinkIO<P>::load_raw(L.gauge, L.gscale, g.V, MU, s);
        const R w8 = R(ph) * LinkIO<P>::scale(L.gscale, s);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          R sc;
          Spinor<R> p = in_raw(r, nf, same, sc);
          if (a.dagger) g5(p);
          Half<R> h = mul_U(u, project<R, MU, -1>(p));
          accum_recon<R, MU, -1>(acc[r], h, w8 * sc);
        }
      }
      // backward: (1 + gamma_mu) U_mu(x - mu)^dag psi(x - mu)
      int nb = neighbour(g, s, tile, tc, lc, MU, -1, &ph, &same);
      if (!a.block || same) {
        SU3<R> u = LinkIO<P>::load_raw(L.gauge, L.gscale, g.V, MU, nb);
        const R w8 = R(ph) * LinkIO<P>::scale(L.gscale, nb);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          R sc;
          Spinor<R> p = in_raw(r, nb, same, sc);
          if (a.dagger) g5(p);
          Half<R> h = mul_Udag(u, project<R, MU, +1>(p));
          accum_recon<R, MU, +1>(acc[r], h, w8 * sc);
        }
      }
    };
    hop(std::integral_constant<int, 0>());
    hop(std::integral_constant<int, 1>());
    hop(std::integral_constant<int, 2>());
    hop(std::integral_constant<int, 3>());

    // clover and the -1/2 of the hopping term; acc becomes the result
    Spinor<R> self[NR];
    R sself[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      self[r] = in_raw(r, s, true, sself[r]);
      if (a.dagger) g5(self[r]);
    }
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      Herm6<R> hc = CloverIO<P>::load_raw(L.clov, L.cscale, g.V, s, blk);
      const R cs = CloverIO<P>::scale(L.cscale, s, blk);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        cplx<R> v[6], o[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) v[i] = self[r].c[2 * blk + i / 3][i % 3];
        herm6_apply(hc, v, o);
        const R w = cs * sself[r];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          cplx<R>& t = acc[r].c[2 * blk + i / 3][i % 3];
          t = w * o[i] - R(0.5) * t;
        }
      }
    }
    double nrm[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (a.dagger) g5(acc[r]);
      if (a.y) {  // residual form: out = y - D in
        Spinor<R> yv = SpinorIO<P>::load(fy[r], s);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < 3; ++c) acc[r].c[i][c] = yv.c[i][c] - acc[r].c[i][c];
      }
      nrm[r] = 0.0;
      const bool skip_r = r >= w.nr || (a.skip && a.skip[L.sys0 + w.rhs0 + r]);
      if (valid && !skip_r) {
        SpinorIO<P>::store(fout[r], s, acc[r]);
        if (a.partials) {
          double t = 0.0;
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c)
              t += double(acc[r].c[i][c].re) * double(acc[r].c[i][c].re) +
                   double(acc[r].c[i][c].im) * double(acc[r].c[i][c].im);
          nrm[r] = t;
        }
      }
    }
    if (a.partials) {
      block_sum<NR>(nrm, red);
      if (threadIdx.x == 0) {
        for (int r = 0; r < w.nr; ++r) a.partials[(size_t)(L.part0 + (w.rhs0 + r) * L.nchunks + w.chunk) * a.pw] = nrm[r];
      }
      __syncthreads();
    }
    if (STAGE) __syncthreads();  // the next item overwrites the staged tile
  }
}

// dynamic LDS of a staged launch: the tile's input spinors (12 complex) and site scale per
// rhs of the lane's tile (nr clamped to the 1..4 the launch switch instantiates)
size_t dirac_stage_lds_bytes(int prec, int nr) {
  const size_t real = prec == P_F64 ? 8 : 4;
  return (2 * real * 12 + real) * (size_t)std::min(std::max(nr, 1), 4) * WG;
}

template <int P, bool S, int PIN>
static void launch_ps(const DiracLaunch& a, int nr, int grid, hipStream_t st) {
  auto lds = [&](int n) { return S ? dirac_stage_lds_bytes(P, n) : size_t(0); };
  switch (nr) {
    case 1: hipLaunchKernelGGL((k_dirac<P, 1, S, PIN>), dim3(grid), dim3(WG), lds(1), st, a); break;
    case 2: hipLaunchKernelGGL((k_dirac<P, 2, S, PIN>), dim3(grid), dim3(WG), lds(2), st, a); break;
    case 3: hipLaunchKernelGGL((k_dirac<P, 3, S, PIN>), dim3(grid), dim3(WG), lds(3), st, a); break;
    default: hipLaunchKernelGGL((k_dirac<P, 4, S, PIN>), dim3(grid), dim3(WG), lds(4), st, a); break;
  }
}

template <int P, int PIN>
static void launch_p(const DiracLaunch& a, int nr, int grid, hipStream_t st) {
  if (a.stage)
    launch_ps<P, true, PIN>(a, nr, grid, st);
  else
    launch_ps<P, false, PIN>(a, nr, grid, st);
}

void launch_dirac(int prec, int nr, const DiracLaunch& a, int grid, hipStream_t st) {
  if (prec == P_F64) {
    switch (a.in_prec) {
      case P_F64: launch_p<P_F64, P_F64>(a, nr, grid, st); break;
      case P_F32: launch_p<P_F64, P_F32>(a, nr, grid, st); break;
      case P_F16: launch_p<P_F64, P_F16>(a, nr, grid, st); break;
      default: launch_p<P_F64, P_BF16>(a, nr, grid, st); break;
    }
    return;
  }
  if (prec == P_F32) {
    switch (a.in_prec) {
      case P_F64: launch_p<P_F32, P_F64>(a, nr, grid, st); break;
      case P_F32: launch_p<P_F32, P_F32>(a, nr, grid, st); break;
      case P_F16: launch_p<P_F32, P_F16>(a, nr, grid, st); break;
      default: launch_p<P_F32, P_BF16>(a, nr, grid, st); break;
    }
    return;
  }
  switch (prec) {
    case P_F16: launch_p<P_F16, P_F16>(a, nr, grid, st); break;
    default: launch_p<P_BF16, P_BF16>(a, nr, grid, st); break;
  }
}

// D_w in FP64 from and to the canonical arrays of the C interface (complex128
// [rhs][lexicographic site][4][3]) in one launch, without a packed copy of the input or of
// the output.  Bound by memory: spinor in and out, links and clover, the neighbours out of
// the chunk and, for several right-hand sides, the operator from the caches.  Against
// pack + k_dirac + unpack: 16^3 x 32 one rhs 78.6 -> 48.6 us a call (40.5 us in the kernel;
// its 201 MB at the rate of a device copy take 41.5), 24^3 x 48 with 12 rhs 3.06 -> 1.74 ms,
// 32^3 x 64 one rhs 0.74 ms (0.66 at the copy rate).
//
// A work-group takes one chunk of WG consecutive sites of the tile-major order and one
// right-hand side, one lane per site; the work-groups of a chunk's right-hand sides are
// neighbours on one XCD, whose L2 serves them the operator.  (Groups of two and three rhs
// sharing a work-group of 512 and 768 lanes were slower: 24^3 x 48 with 12 rhs 1.76 / 2.05 /
// 2.16 ms, 16^3 x 32 with two rhs 56 / 65 us.)  The chunk's spinors are staged in LDS: a
// canonical site is 192 contiguous bytes, so the copy runs over (site, component) with the
// component fastest (runs of B3 sites are contiguous) and the lanes then read component rows;
// rows are one element longer than the chunk, which spreads the copy's 12 rows over the LDS
// banks.  Hops inside the chunk read LDS, the others gather 192 contiguous bytes from the
// canonical array.  The result goes back through the same LDS rows, with non-temporal stores
// (the output then does not displace the input: 12 rhs 1.76 -> 1.74 ms, 32^3 x 64 0.77 -> 0.74).
constexpr int DC_ROW = WG + 1;

// Loads of this kernel: a uniform base (pointer and row, kept in scalar registers) plus one
// 32-bit byte offset per site, so that the rows of a link or clover block share one address
// register (16 bytes x V < 4 GiB: a lattice of 2^28 sites would not fit the GPU's memory).
WC_D gd2v ld_row(const void* base, size_t row, unsigned off) {
  return *(gptr_t<gd2v>)((const __attribute__((address_space(1))) char*)base + row * 16 + off);
}
WC_D SU3<double> canon_link(const void* gauge, int V, int mu, unsigned off) {
  SU3<double> u;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const gd2v v = ld_row(gauge, (size_t)(mu * 9 + k) * V, off);
    u.m[k / 3][k % 3] = {v.x, v.y};
  }
  return u;
}
WC_D Herm6<double> canon_clover(const void* clov, int V, int blk, unsigned off) {
  Herm6<double> h;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const gd2v v = ld_row(clov, (size_t)(18 * blk + k) * V, off);
    h.d[2 * k] = v.x;
    h.d[2 * k + 1] = v.y;
  }
#pragma unroll
  for (int k = 0; k < 15; ++k) {
    const gd2v v = ld_row(clov, (size_t)(18 * blk + 3 + k) * V, off);
    h.o[k] = {v.x, v.y};
  }
  return h;
}

__global__ __launch_bounds__(WG) void k_dirac_canon(DiracCanonLaunch a) {
  typedef double R;
  extern __shared__ double stage_d[];
  double2* st = (double2*)stage_d;       // [12][DC_ROW]
  int* lexs = (int*)(st + 12 * DC_ROW);  // [WG] canonical site indices
  const Geom& g = a.g;
  const int it = xcd_remap(blockIdx.x, gridDim.x);
  const int chunk = it / a.nrhs, r = it - chunk * a.nrhs;
  const int t = threadIdx.x;
  const int s0 = chunk * WG;
  const bool valid = s0 + t < g.V;
  const int s = valid ? s0 + t : g.V - 1;
  const int tile = s / g.bvol;
  int tc[4], lc[4], x[4];
  tile_coords(g, tile, tc);
  local_coords(g, s - tile * g.bvol, lc);
#pragma unroll
  for (int m = 0; m < 4; ++m) x[m] = tc[m] * g.B[m] + lc[m];
  const int lex = ((x[0] * g.L[1] + x[1]) * g.L[2] + x[2]) * g.L[3] + x[3];
  lexs[t] = lex;
  const double2* in = a.in + (size_t)r * g.V * 12;
  __syncthreads();
  const int nel = (s0 + WG <= g.V ? WG : g.V - s0) * 12;
#pragma unroll
  for (int j = 0; j < 12; ++j) {
    const int e = j * WG + t;
    if (e < nel) {
      const int site = e / 12, k = e - site * 12;
      st[k * DC_ROW + site] = gld_d2(in, (size_t)lexs[site] * 12 + k);
    }
  }
  __syncthreads();

  // input spinor at the site with internal index n and canonical index nlex
  auto input = [&](int n, int nlex) {
    Spinor<R> p;
    const unsigned ln = (unsigned)(n - s0);
    if (ln < (unsigned)WG) {
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const double2 v = st[k * DC_ROW + ln];
        p.c[k / 3][k % 3] = {v.x, v.y};
      }
    } else {
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const double2 v = gld_d2(in, (size_t)nlex * 12 + k);
        p.c[k / 3][k % 3] = {v.x, v.y};
      }
    }
    if (a.dagger) g5(p);
    return p;
  };

  Spinor<R> acc;
  zero(acc);
  if (valid) {
    auto hop = [&](auto MUc) {
      constexpr int MU = decltype(MUc)::value;
      const int stride = MU == 3 ? 1 : MU == 2 ? g.L[3] : MU == 1 ? g.L[3] * g.L[2] : g.L[3] * g.L[2] * g.L[1];
      const int wrap = (g.L[MU] - 1) * stride;
      int ph;
      bool same;
      const int nf = neighbour(g, s, tile, tc, lc, MU, +1, &ph, &same);
      if (!a.block || same) {
        const SU3<R> u = canon_link(a.gauge, g.V, MU, 16u * s);
        const Spinor<R> p = input(nf, x[MU] + 1 < g.L[MU] ? lex + stride : lex - wrap);
        accum_recon<R, MU, -1>(acc, mul_U(u, project<R, MU, -1>(p)), R(ph));
      }
      const int nb = neighbour(g, s, tile, tc, lc, MU, -1, &ph, &same);
      if (!a.block || same) {
        const SU3<R> u = canon_link(a.gauge, g.V, MU, 16u * nb);
        const Spinor<R> p = input(nb, x[MU] > 0 ? lex - stride : lex + wrap);
        accum_recon<R, MU, +1>(acc, mul_Udag(u, project<R, MU, +1>(p)), R(ph));
      }
    };
    hop(std::integral_constant<int, 0>());
    hop(std::integral_constant<int, 1>());
    hop(std::integral_constant<int, 2>());
    hop(std::integral_constant<int, 3>());

    // clover and the -1/2 of the hopping term; acc becomes the result
    const Spinor<R> self = input(s, lex);
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      const Herm6<R> hc = canon_clover(a.clov, g.V, blk, 16u * s);
      cplx<R> v[6], o[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) v[i] = self.c[2 * blk + i / 3][i % 3];
      herm6_apply(hc, v, o);
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        cplx<R>& q = acc.c[2 * blk + i / 3][i % 3];
        q = o[i] - R(0.5) * q;
      }
    }
    if (a.dagger) g5(acc);
  }
  __syncthreads();  // every lane has read the staged input
  if (valid) {
#pragma unroll
    for (int k = 0; k < 12; ++k)
      st[k * DC_ROW + t] = make_double2(acc.c[k / 3][k % 3].re, acc.c[k / 3][k % 3].im);
  }
  __syncthreads();
  double2* out = a.out + (size_t)r * g.V * 12;
#pragma unroll
  for (int j = 0; j < 12; ++j) {
    const int e = j * WG + t;
    if (e < nel) {
      const int site = e / 12, k = e - site * 12;
      const double2 v = st[k * DC_ROW + site];
      __builtin_nontemporal_store(gd2v{v.x, v.y}, (gd2v*)(out + (size_t)lexs[site] * 12 + k));
    }
  }
}

void launch_dirac_canon(const DiracCanonLaunch& a, hipStream_t st) {
  const int nchunks = (a.g.V + WG - 1) / WG;
  const size_t lds = sizeof(double2) * 12 * DC_ROW + sizeof(int) * WG;
  hipLaunchKernelGGL(k_dirac_canon, dim3((unsigned)nchunks * a.nrhs), dim3(WG), lds, st, a);
}

}  // namespace wc
