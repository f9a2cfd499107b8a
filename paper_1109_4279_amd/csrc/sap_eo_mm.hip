// Even/odd-preconditioned block solver (arXiv:1109.4279, Sec. 4, Table 1) for several
// right-hand sides on the matrix cores, 16-bit storage, FP32 arithmetic.
//
// The same solve as k_sap_eo: MR on S = A_ee - H_eo A_oo^-1 H_oe on the even half of a block,
// then the odd half.  Every product of it is a complex 3x3 matrix (a link, or one of the four
// colour blocks of a 6x6 clover block) times colour vectors, and with four right-hand sides
// the matrix has four vectors: v_mfma_f32_4x4x1 holds 16 independent 4x4 products, so one
// instruction advances 16 sites by one column of the matrix.
//
// Work mapping: one work-group per (block, up to four rhs).  A wavefront takes 16 site pairs
// (one even, one odd site); lane l holds rhs l % 4 of pair l / 4, all 12 components of it.
// As matrix operand the lane supplies row l % 4 of its site's matrix (rows 0..2; row 3 of the
// product is never read), as vector operand its own component, and it receives its own
// product: projection, reconstruction and the MR recursion stay within the lane.  A 3x3
// complex product is 12 instructions (three columns, real and imaginary part of both).
//
// What bounds it: issue.  k_sap_eo issues 1957 vector instructions per wavefront of 64
// (site, rhs) and MR step, two thirds of them the FMAs of these products and the decoding of
// the operator per rhs; here a wavefront issues 1257 vector and 576 matrix instructions for 128
// of them (SQ_INSTS_VALU, which counts both, and SQ_INSTS_MFMA, launches of 4 steps less launches
// of none).  A 4x4x1 matrix instruction holds its SIMD for 8 cycles (SQ_VALU_MFMA_BUSY_CYCLES),
// a vector one for 4, and vector instructions do not run beside it: with two wavefronts per SIMD a
// step of a block takes 22 100 cycles against 19 300 of issue (87 %; set-up and stores 33 %).
// 24^3 x 48, 12 rhs, BF16: half-sweep 1460 (k_sap_eo) -> 1067 us, of it set-up and stores
// 507 us, an MR step 140 us (214 us).  (With the matrix instructions in runs of 24 instead of
// 48, see mm_hops, and the field addresses spilled over the MR loop: 1213 us.)
//
// Operator: the block's links are staged in LDS once (9 packed words each); the lane's rows
// of the two clover blocks of its two sites are kept packed in registers (48 words).  The
// vectors are exchanged through LDS slots (even sites first, then odd, then one slot of
// zeros that stands for every neighbour outside the block): 4 rhs x 12 components at a stride
// of 448 bytes, which puts four consecutive slots on distinct
// banks.  115 KB + 37 KB for a 256-site block: one work-group of 8 wavefronts per CU, with
// 256 registers per lane.
//
// The odd half of the solution is accumulated along the MR steps: z_o = A_oo^-1 eta_o -
// sum_k alpha_k A_oo^-1 H_oe rho_k, whose terms each step has in LDS anyway, so that the
// last application of H_oe and A_oo^-1 falls away.
#include "wc_kernels.h"

namespace wc {

constexpr int MM_SLOT = 448;       // bytes of an exchange slot: [6][4 rhs] float4 and padding
constexpr int MM_ENT = 192;        // bytes of a border entry: [3][4 rhs] float4
constexpr int MM_MAX_WAVES = 8;

typedef float mf4 __attribute__((ext_vector_type(4)));

// one complex 3x3 matrix row as the lane's matrix operand: re, im and -im of three columns
struct MRow {
  float re[3], im[3], ni[3];
};

// the row from its packed words (CONJ: of the complex conjugate)
template <int P, bool CONJ = false> WC_D void unpack_row(const uint32_t* w, MRow& r) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float im;
    if constexpr (P == P_BF16) {
      r.re[k] = __uint_as_float(w[k] << 16);
      im = __uint_as_float(w[k] & 0xFFFF0000u);
    } else {
      r.re[k] = s16_to_f32<P>(uint16_t(w[k] & 0xFFFFu));
      im = s16_to_f32<P>(uint16_t(w[k] >> 16));
    }
    r.im[k] = CONJ ? -im : im;
    r.ni[k] = CONJ ? im : -im;
  }
}

// (cre, cim) += M v, M by rows over the lanes of the site, v this lane's colour vector.
// Every lane of the wavefront executes this (the matrix instructions ignore the lane mask).
WC_D void mm3(const MRow& m, const cplx<float>* v, mf4& cre, mf4& cim) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    cre = __builtin_amdgcn_mfma_f32_4x4x1f32(m.re[k], v[k].re, cre, 0, 0, 0);
    cim = __builtin_amdgcn_mfma_f32_4x4x1f32(m.im[k], v[k].re, cim, 0, 0, 0);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    cre = __builtin_amdgcn_mfma_f32_4x4x1f32(m.ni[k], v[k].im, cre, 0, 0, 0);
    cim = __builtin_amdgcn_mfma_f32_4x4x1f32(m.re[k], v[k].im, cim, 0, 0, 0);
  }
}

WC_D Half<float> mm_half(const MRow& m, const Half<float>& h) {
  Half<float> t;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    mf4 cre = {0.f, 0.f, 0.f, 0.f}, cim = {0.f, 0.f, 0.f, 0.f};
    mm3(m, h.c[s], cre, cim);
#pragma unroll
    for (int a = 0; a < 3; ++a) t.c[s][a] = {cre[a], cim[a]};
  }
  return t;
}

// acc += w x (the reconstruction of the transported half spinor t), as fused multiply-adds
template <int MU, int SGN> WC_D void recon_fma(Spinor<float>& acc, const Half<float>& t, float w) {
  auto add = [&](cplx<float>& a, float c, cplx<float> x) { a = {fmaf(c, x.re, a.re), fmaf(c, x.im, a.im)}; };
  auto addi = [&](cplx<float>& a, float c, cplx<float> x) { a = {fmaf(-c, x.im, a.re), fmaf(c, x.re, a.im)}; };
  const float p = SGN > 0 ? w : -w;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cplx<float> t0 = t.c[0][a], t1 = t.c[1][a];
    add(acc.c[0][a], w, t0);
    add(acc.c[1][a], w, t1);
    if (MU == 0) {  // lower = -SGN t
      add(acc.c[2][a], -p, t0);
      add(acc.c[3][a], -p, t1);
    } else if (MU == 1) {  // SGN (i t1, i t0)
      addi(acc.c[2][a], p, t1);
      addi(acc.c[3][a], p, t0);
    } else if (MU == 2) {  // SGN (t1, -t0)
      add(acc.c[2][a], p, t1);
      add(acc.c[3][a], -p, t0);
    } else {  // SGN (i t0, -i t1)
      addi(acc.c[2][a], p, t0);
      addi(acc.c[3][a], -p, t1);
    }
  }
}

template <int P> WC_D Spinor<float> unpack_spinor(const uint4* v) {
  Spinor<float> o;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = 4 * k + i;
      o.c[c / 3][c % 3] = {s16_to_f32<P>(uint16_t(w[i] & 0xFFFFu)), s16_to_f32<P>(uint16_t(w[i] >> 16))};
    }
  }
  return o;
}

WC_D Spinor<float> slot_read(const char* q) {
  Spinor<float> p;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const mf4 v = *(const mf4*)(q + 64 * k);
    p.c[(2 * k) / 3][(2 * k) % 3] = {v.x, v.y};
    p.c[(2 * k + 1) / 3][(2 * k + 1) % 3] = {v.z, v.w};
  }
  return p;
}
WC_D void slot_write(char* q, const Spinor<float>& p) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const cplx<float> a = p.c[(2 * k) / 3][(2 * k) % 3], b = p.c[(2 * k + 1) / 3][(2 * k + 1) % 3];
    *(mf4*)(q + 64 * k) = mf4{a.re, a.im, b.re, b.im};
  }
}

// The hops into one site from inside the block, times wt: nb holds the slots of its eight
// neighbours (two per word, direction by direction, forward first), own its own slot, ls the
// slot of zeros.
template <int P>
WC_D Spinor<float> mm_hops(const char* xch, const uint32_t* lk, const float* lsc, int ls, const uint32_t* nb, int own,
                           int j, int jr, float wt) {
  const int lrow = ls + 1;
  Spinor<float> acc;
  zero(acc);
  const float w_own = wt * lsc[own];
  // Both hops of a direction are projected, multiplied and reconstructed together: matrix and
  // vector instructions that alternate on a SIMD, of one wavefront or of two, cost about 9
  // cycles more per alternation than one after the other, so the matrix instructions come in
  // runs of 48.  (Measured: 24 matrix + 48 vector instructions in turn on two wavefronts 1037
  // cycles, 48 + 96 in turn 900 for the same work, the sum of the parts 864.)
  auto dir = [&](auto MUc) {
    constexpr int MU = decltype(MUc)::value;
    const int sf = nb[MU] & 0xFFFFu, sb = nb[MU] >> 16;
    const uint32_t* lf = lk + (MU * lrow + own) * 9 + 3 * jr;
    const uint32_t* lb = lk + (MU * lrow + sb) * 9 + jr;  // rows of U^dag: columns of U, conjugated
    const uint32_t wf[3] = {lf[0], lf[1], lf[2]}, wb[3] = {lb[0], lb[3], lb[6]};
    MRow mf, mb;
    const Half<float> hf = project<float, MU, -1>(slot_read(xch + sf * MM_SLOT + 16 * j));
    const Half<float> hb = project<float, MU, +1>(slot_read(xch + sb * MM_SLOT + 16 * j));
    const float w_b = wt * lsc[sb];
    unpack_row<P>(wf, mf);
    unpack_row<P, true>(wb, mb);
    __builtin_amdgcn_sched_barrier(0);
    const Half<float> tf = mm_half(mf, hf), tb = mm_half(mb, hb);
    __builtin_amdgcn_sched_barrier(0);
    recon_fma<MU, -1>(acc, tf, w_own);
    recon_fma<MU, +1>(acc, tb, w_b);
    __builtin_amdgcn_sched_barrier(0);
  };
  dir(std::integral_constant<int, 0>());
  dir(std::integral_constant<int, 1>());
  dir(std::integral_constant<int, 2>());
  dir(std::integral_constant<int, 3>());
  return acc;
}

// This lane's rows of a site's clover blocks, packed: [chirality][2 s + s'][column]
struct ClRows {
  uint32_t w[2][4][3];
  float sc[2];
};

// (clov_mm holds them ready: [chirality][2 s + s'][V][row][column])
WC_D void clover_rows(const LatDesc& L, int site, int jr, ClRows& c) {
  const size_t V = L.g.V;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      typedef uint32_t u3 __attribute__((ext_vector_type(3), aligned(4)));
      const u3 v = *(gptr_t<u3>)((gptr_t<uint32_t>)L.clov_mm + (4 * b + m) * V * 9 + (unsigned)(site * 9 + 3 * jr));
      c.w[b][m][0] = v.x;
      c.w[b][m][1] = v.y;
      c.w[b][m][2] = v.z;
    }
  c.sc[0] = gld_f(L.cscale_eo, 2 * (size_t)site);
  c.sc[1] = gld_f(L.cscale_eo, 2 * (size_t)site + 1);
}

// Keeps the words packed: without it the compiler unpacks them once ahead of the MR loop,
// into twice the registers, and spills.
WC_D void keep_packed(ClRows& c) {
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(c.w[b][i][k]));
}

// C v without the block scales
template <int P> WC_D Spinor<float> mm_clover(const ClRows& c, const Spinor<float>& v) {
  Spinor<float> o;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    MRow m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) unpack_row<P>(c.w[b][i], m[i]);
    __builtin_amdgcn_sched_barrier(0);
    mf4 cre[2], cim[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      cre[s] = cim[s] = mf4{0.f, 0.f, 0.f, 0.f};
      mm3(m[2 * s], v.c[2 * b], cre[s], cim[s]);
      mm3(m[2 * s + 1], v.c[2 * b + 1], cre[s], cim[s]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int a = 0; a < 3; ++a) o.c[2 * b + s][a] = {cre[s][a], cim[s][a]};
  }
  return o;
}

// sum over the 16 lanes of a wavefront that hold the same rhs (lane % 4); every lane gets it
WC_D float rhs_sum(float v) {
  v += dpp_mov<0x124>(v);  // row_ror 4
  v += dpp_mov<0x128>(v);  // row_ror 8: all four lanes of this rhs in the 16-lane row
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

template <int P>
__global__ __launch_bounds__(64 * MM_MAX_WAVES, 2) void k_sap_eo_mm(SapLaunch a) {
  extern __shared__ __align__(16) char smem[];
  const WorkItem w = load_uniform(a.items, xcd_remap(blockIdx.x, a.nitems));
  const LatDesc L = load_uniform(a.lats, w.lat);
  const Geom& g = L.g;
  bool any = true;
  if (a.skip) {
    any = false;
    for (int r = 0; r < w.nr; ++r) any |= (a.skip[L.sys0 + w.rhs0 + r] == 0);
  }
  if (!any) return;
  const int nh = (g.bvol + 1) >> 1, ls = 2 * nh, lrow = ls + 1;
  char* xch = smem;                                       // [ls + 1] slots, or the border entries
  uint32_t* lk = (uint32_t*)(smem + a.mm_xch_bytes);      // [4][ls + 1][9] packed links
  mf4* red = (mf4*)(lk + 4 * lrow * 9);                    // [MM_MAX_WAVES][4 rhs]
  float* lsc = (float*)(red + MM_MAX_WAVES * 4);          // [ls + 1] link scales

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  const int j = lane & 3, jr = j < 3 ? j : 2;
  const int pr = wave * 16 + (lane >> 2);
  const int tile = __builtin_amdgcn_readfirstlane(gld_i32(a.colour ? L.tiles[1] : L.tiles[0], w.chunk));
  const int base = tile * g.bvol;
  int tc[4];
  tile_coords(g, tile, tc);
  const int cp = (tc[0] * g.B[0] + tc[1] * g.B[1] + tc[2] * g.B[2] + tc[3] * g.B[3]) & 1;
  const int le = pr < nh ? gld_s16(L.eo_sites, (2 * cp) * nh + pr) : -1;
  const int lo = pr < nh ? gld_s16(L.eo_sites, (2 * cp + 1) * nh + pr) : -1;
  const bool he = le >= 0, ho = lo >= 0;
  const int lel = he ? le : 0, lol = ho ? lo : 0;
  const int se = base + lel, so = base + lol;
  // slots: a lane without a site works on the slot of zeros and writes nothing
  const int we = he ? pr : ls, wo = ho ? nh + pr : ls;
  uint32_t nbe[4], nbo[4];
  {
    const uint4 e = gld_u4(L.eo_nbr, cp * g.bvol + lel), o = gld_u4(L.eo_nbr, cp * g.bvol + lol);
    const uint32_t zz = ls | (ls << 16);
    nbe[0] = he ? e.x : zz; nbe[1] = he ? e.y : zz; nbe[2] = he ? e.z : zz; nbe[3] = he ? e.w : zz;
    nbo[0] = ho ? o.x : zz; nbo[1] = ho ? o.y : zz; nbo[2] = ho ? o.z : zz; nbo[3] = ho ? o.w : zz;
  }
  const bool live = j < w.nr;
  const bool store = live && !(a.skip && a.skip[L.sys0 + w.rhs0 + (live ? j : 0)]);
  // this lane's rhs in a field
  auto field = [&](void* d, float* sc, int lane_rhs) {
    const long long off = L.foff + (long long)(w.rhs0 + lane_rhs) * g.V;
    return FieldRef{(char*)d + off * 48, sc + off, g.V};
  };
  const FieldRef frho = field(a.rho, a.rho_sc, live ? j : 0);
  const FieldRef fz = field(a.z, a.z_sc, live ? j : 0);

  // Everything the set-up reads is requested before the first use (one work-group per CU
  // leaves nothing else to cover the latency): residual, links and clover rows.
  Spinor<float> ve = SpinorIO<P>::load(frho, se), vo;
  if (a.odd_rho == 2)
    zero(vo);
  else
    vo = SpinorIO<P>::load(frho, so);
  // the block's links and their scales; the slot of zeros has zero links
  for (int i = threadIdx.x; i < 4 * g.bvol; i += blockDim.x) {
    const int mu = i / g.bvol, l = i - mu * g.bvol;
    const int slot = gld_s16(L.eo_slot, cp * g.bvol + l);
    const size_t p = (size_t)mu * 2 * g.V + base + l;
    const uint4 x = gld_u4(L.gauge, p), y = gld_u4(L.gauge, p + g.V);
    const uint32_t z = gld_u32(L.gauge, (size_t)8 * g.V * 4 + (size_t)mu * g.V + base + l);
    uint32_t* q = lk + (mu * lrow + slot) * 9;
    q[0] = x.x; q[1] = x.y; q[2] = x.z; q[3] = x.w;
    q[4] = y.x; q[5] = y.y; q[6] = y.z; q[7] = y.w;
    q[8] = z;
    if (mu == 0) lsc[slot] = gld_f(L.gscale, base + l);
  }
  if (threadIdx.x < 4 * 9) lk[((threadIdx.x / 9) * lrow + ls) * 9 + threadIdx.x % 9] = 0;
  if (threadIdx.x == 0) lsc[ls] = 0.f;
  // bring the residual up to date with the other colour's latest block solutions
  if (a.border) {
    const uint4 gte = gld_u4(L.eo_bgat, lel), gto = gld_u4(L.eo_bgat, lol);
    const int ne = border_entry_count(g.B);
    const int rounds = (ne + 16 * nwaves - 1) / (16 * nwaves);
    constexpr int UN = 4;  // rounds whose loads are in flight together (all of a 4^4 block's)
    for (int rd = 0; rd < rounds; rd += UN) {
      uint32_t rw[UN][3], dd[UN];
      uint4 raw[UN][3];
      float wgt[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int e = ((rd + u) * nwaves + wave) * 16 + (lane >> 2);
        const uint32_t ent = gld_u32(L.eo_bent, e < ne ? e : 0);
        const int local = ent & 0xFFu, nl = (ent >> 8) & 0xFFu, d = (ent >> 16) & 7u;
        const int mu = d >> 1;
        const bool fwd = (d & 1) == 0;
        const int nb_mu = mu == 0 ? g.NB[0] : mu == 1 ? g.NB[1] : mu == 2 ? g.NB[2] : g.NB[3];
        const int ts = mu == 0 ? g.tstr[0] : mu == 1 ? g.tstr[1] : mu == 2 ? g.tstr[2] : g.tstr[3];
        const int tm = mu == 0 ? tc[0] : mu == 1 ? tc[1] : mu == 2 ? tc[2] : tc[3];
        const bool wrap = fwd ? tm + 1 == nb_mu : tm == 0;
        const int nt = tile + (fwd ? (wrap ? -(nb_mu - 1) * ts : ts) : (wrap ? (nb_mu - 1) * ts : -ts));
        const int ns = nt * g.bvol + nl;
        const float ph = (wrap && mu == 0) ? float(g.bc_t) : 1.f;
        const int lsite = fwd ? base + local : ns;  // the site whose link the hop crosses
        // this lane's row: words 3 jr .. of U, or words jr, jr + 3, jr + 6 of U, conjugated
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int n = fwd ? 3 * jr + k : jr + 3 * k;
          const size_t at = n < 8 ? ((size_t)(2 * mu + (n >> 2)) * g.V + lsite) * 4 + (n & 3)
                                  : (size_t)8 * g.V * 4 + (size_t)mu * g.V + lsite;
          const uint32_t v = gld_u32(L.gauge, at);
          rw[u][k] = fwd ? v : v ^ 0x80000000u;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) raw[u][k] = gld_u4(fz.d, (size_t)k * g.V + ns);
        wgt[u] = 0.5f * ph * LinkIO<P>::scale(L.gscale, lsite) * SpinorIO<P>::scale(fz, ns);
        dd[u] = d;
      }
#pragma unroll
      for (int v = 0; v < UN; v += 2) {  // two rounds' products together
        Half<float> h[UN];
        MRow m[UN];
#pragma unroll
        for (int u = v; u < v + 2; ++u) {
          const Spinor<float> p = unpack_spinor<P>(raw[u]);
          switch (dd[u]) {
            case 0: h[u] = project<float, 0, -1>(p); break;
            case 1: h[u] = project<float, 0, +1>(p); break;
            case 2: h[u] = project<float, 1, -1>(p); break;
            case 3: h[u] = project<float, 1, +1>(p); break;
            case 4: h[u] = project<float, 2, -1>(p); break;
            case 5: h[u] = project<float, 2, +1>(p); break;
            case 6: h[u] = project<float, 3, -1>(p); break;
            default: h[u] = project<float, 3, +1>(p); break;
          }
          unpack_row<P>(rw[u], m[u]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = v; u < v + 2; ++u) h[u] = mm_half(m[u], h[u]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = v; u < v + 2; ++u) {
          const int e = ((rd + u) * nwaves + wave) * 16 + (lane >> 2);
          if (e >= ne) continue;
          char* q = xch + (size_t)e * MM_ENT + 16 * j;
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const cplx<float> x = h[u].c[(2 * k) / 3][(2 * k) % 3], y = h[u].c[(2 * k + 1) / 3][(2 * k + 1) % 3];
            *(mf4*)(q + 64 * k) = mf4{wgt[u] * x.re, wgt[u] * x.im, wgt[u] * y.re, wgt[u] * y.im};
          }
        }
      }
    }
    __syncthreads();
    auto gather = [&](const uint4& gt, Spinor<float>& v) {
      const uint32_t gw[4] = {gt.x, gt.y, gt.z, gt.w};
      auto one = [&](auto MUc, auto SGNc, int e) {
        if (e == 0xFFFF) return;
        const char* q = xch + (size_t)e * MM_ENT + 16 * j;
        Half<float> t;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const mf4 x = *(const mf4*)(q + 64 * k);
          t.c[(2 * k) / 3][(2 * k) % 3] = {x.x, x.y};
          t.c[(2 * k + 1) / 3][(2 * k + 1) % 3] = {x.z, x.w};
        }
        recon_fma<decltype(MUc)::value, decltype(SGNc)::value>(v, t, 1.f);
      };
      auto both = [&](auto MUc) {
        constexpr int MU = decltype(MUc)::value;
        one(MUc, std::integral_constant<int, -1>(), int(gw[MU] & 0xFFFFu));
        one(MUc, std::integral_constant<int, +1>(), int(gw[MU] >> 16));
      };
      both(std::integral_constant<int, 0>());
      both(std::integral_constant<int, 1>());
      both(std::integral_constant<int, 2>());
      both(std::integral_constant<int, 3>());
    };
    gather(gte, ve);
    gather(gto, vo);
    __syncthreads();  // the entries' space becomes the exchange slots
  }

  ClRows ce, co;
  clover_rows(L, so, jr, co);
  clover_rows(L, se, jr, ce);
  for (int i = threadIdx.x; i < MM_SLOT / 4; i += blockDim.x) ((float*)(xch + ls * MM_SLOT))[i] = 0.f;

  // z_o = A_oo^-1 eta_o to start with; source of the Schur system: eta_e - H_eo z_o
  Spinor<float> zo = mm_clover<P>(co, vo);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) zo.c[i][c] = co.sc[i / 2] * zo.c[i][c];
  char* const my_e = xch + we * MM_SLOT + 16 * j;
  char* const my_o = xch + wo * MM_SLOT + 16 * j;
  if (ho) slot_write(my_o, zo);
  __syncthreads();
  {
    const Spinor<float> d = mm_hops<P>(xch, lk, lsc, ls, nbe, we, j, jr, 0.5f);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) ve.c[i][c] = ve.c[i][c] + d.c[i][c];
  }
  if (he) slot_write(my_e, ve);

  Spinor<float> ze;
  zero(ze);
  for (int it = 0; it < a.nmr; ++it) {
    keep_packed(ce);
    keep_packed(co);
    // q = A_ee rho - H_eo A_oo^-1 H_oe rho  (H = -1/2 sum of hops), rho in the even slots
    __syncthreads();
    {
      const Spinor<float> t = mm_hops<P>(xch, lk, lsc, ls, nbo, wo, j, jr, -0.5f);
      Spinor<float> u = mm_clover<P>(co, t);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) u.c[i][c] = co.sc[i / 2] * u.c[i][c];
      if (ho) slot_write(my_o, u);
    }
    __syncthreads();
    Spinor<float> q = mm_hops<P>(xch, lk, lsc, ls, nbe, we, j, jr, 0.5f);
    Spinor<float> rho = slot_read(my_e);
    {
      const Spinor<float> t = mm_clover<P>(ce, rho);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c)
          q.c[i][c] = {fmaf(ce.sc[i / 2], t.c[i][c].re, q.c[i][c].re), fmaf(ce.sc[i / 2], t.c[i][c].im, q.c[i][c].im)};
    }
    float qre = 0.f, qim = 0.f, qq = 0.f;
    if (he) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const cplx<float> x = q.c[i][c], y = rho.c[i][c];
          qre += x.re * y.re + x.im * y.im;
          qim += x.re * y.im - x.im * y.re;
          qq += x.re * x.re + x.im * x.im;
        }
    }
    qre = rhs_sum(qre);
    qim = rhs_sum(qim);
    qq = rhs_sum(qq);
    if (lane < 4) red[wave * 4 + j] = mf4{qre, qim, qq, 0.f};
    __syncthreads();
    double s0 = 0, s1 = 0, s2 = 0;
    for (int v = 0; v < nwaves; ++v) {
      const mf4 x = red[v * 4 + j];
      s0 += double(x.x);
      s1 += double(x.y);
      s2 += double(x.z);
    }
    const cplx<float> alpha = {float(s2 > 0.0 ? s0 / s2 : 0.0), float(s2 > 0.0 ? s1 / s2 : 0.0)};
    const Spinor<float> u = slot_read(my_o);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        cmac(ze.c[i][c], alpha, rho.c[i][c]);
        cmac(zo.c[i][c], -alpha, u.c[i][c]);  // u = A_oo^-1 H_oe rho
        ve.c[i][c] = rho.c[i][c];
        cmac(ve.c[i][c], -alpha, q.c[i][c]);
      }
    if (he) slot_write(my_e, ve);
  }

  if (!store) return;
  // (the field addresses anew: kept from the set-up they would spill over the MR loop)
  int jl = j;
  asm volatile("" : "+v"(jl));
  const FieldRef orho = field(a.rho, a.rho_sc, jl), oz = field(a.z, a.z_sc, jl), fpsi = field(a.psi, a.psi_sc, jl);
  Spinor<float> pe, po;
  zero(pe);
  zero(po);
  if (!a.first) {
    pe = SpinorIO<P>::load(fpsi, se);
    po = SpinorIO<P>::load(fpsi, so);
  }
  auto put = [&](int site, const Spinor<float>& z, const Spinor<float>& res, const Spinor<float>& psi, bool wr) {
    if (wr) SpinorIO<P>::store(orho, site, res);
    if (a.write_z) SpinorIO<P>::store(oz, site, z);
    Spinor<float> p = z;
    if (!a.first) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) p.c[i][c] = z.c[i][c] + psi.c[i][c];
    }
    SpinorIO<P>::store(fpsi, site, p);
  };
  if (he) put(se, ze, ve, pe, a.write_rho);
  if (ho) {
    Spinor<float> none;
    zero(none);
    put(so, zo, none, po, a.write_rho && a.odd_rho == 0);
  }
}

// The rows of every site's even/odd clover blocks as the lanes take them: block (s, s') of a
// chirality by rows of three packed complex entries, below the diagonal the conjugate.  A
// stored chirality block has 3 words of two diagonal entries, then the 15 above the diagonal.
__global__ __launch_bounds__(WG) void k_clover_mm(int V, const uint32_t* src, uint32_t* dst) {
  const int s = blockIdx.x * WG + threadIdx.x;
  if (s >= V) return;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    uint32_t w[18];
#pragma unroll
    for (int n = 0; n < 18; ++n) {
      const int q = 18 * b + n;
      w[n] = src[((size_t)(q >> 2) * V + s) * 4 + (q & 3)];
    }
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int m = 0; m < 6; ++m) {
        const int lo = i < m ? i : m, hi = i < m ? m : i;
        uint32_t v;
        if (i == m)
          v = (i & 1) ? w[i >> 1] >> 16 : w[i >> 1] & 0xFFFFu;
        else
          v = w[3 + lo * (11 - lo) / 2 + hi - lo - 1] ^ (i > m ? 0x80000000u : 0u);
        dst[(((size_t)(4 * b + 2 * (i / 3) + m / 3) * V + s) * 3 + i % 3) * 3 + m % 3] = v;
      }
  }
}

void launch_clover_mm(int V, const void* clov_eo16, void* dst, hipStream_t st) {
  hipLaunchKernelGGL(k_clover_mm, dim3((V + WG - 1) / WG), dim3(WG), 0, st, V, (const uint32_t*)clov_eo16,
                     (uint32_t*)dst);
}

int sap_eo_mm_waves(int bvol) { return ((bvol + 1) / 2 + 15) / 16; }

size_t sap_eo_mm_xch_bytes(int bvol, int border_entries) {
  const size_t slots = (size_t)(2 * ((bvol + 1) / 2) + 1) * MM_SLOT;
  const size_t ents = (size_t)border_entries * MM_ENT;
  return slots > ents ? slots : ents;
}
size_t sap_eo_mm_lds_bytes(int bvol, int border_entries) {
  const size_t links = (size_t)4 * (2 * ((bvol + 1) / 2) + 1) * 9 * 4;
  return sap_eo_mm_xch_bytes(bvol, border_entries) + (links + 15) / 16 * 16 + (size_t)MM_MAX_WAVES * 4 * 16 +
         sizeof(float) * (2 * ((bvol + 1) / 2) + 1);
}

void launch_sap_eo_mm(int prec, const SapLaunch& a, int bvol, int border_entries, hipStream_t st) {
  const size_t lds = sap_eo_mm_lds_bytes(bvol, border_entries);
  const int threads = 64 * sap_eo_mm_waves(bvol);
  if (prec == P_F16)
    hipLaunchKernelGGL((k_sap_eo_mm<P_F16>), dim3(a.nitems), dim3(threads), lds, st, a);
  else
    hipLaunchKernelGGL((k_sap_eo_mm<P_BF16>), dim3(a.nitems), dim3(threads), lds, st, a);
}

}  // namespace wc
