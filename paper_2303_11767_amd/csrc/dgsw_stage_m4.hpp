// One stage of the DG right-hand side at r = 3 in FP64 on the matrix cores.
//
// At r = 3 every 1-D table of the sum-factorised stage is a 4 x 4 matrix, so
// each contraction of an element is one block of v_mfma_f64_4x4x4_4b: four
// independent products D = A B + C per wavefront, one element each.  Lane l
// belongs to element (l / 4) % 4 and holds entry (x, y) = (l / 16, l % 4) of
// every 4 x 4 array of that element.  The operand layouts are A[i = y][k = x],
// B[k = x][j = y], D[i = x][j = y]: a result used as B is itself, used as A
// its transpose, so
//     mfma(X, T) = X^T T   (contracts the x index of X with the table T)
//     mfma(T, X) = T^T X   (contracts the x index of X from the left)
// and applying the first twice turns modes [b][a] into nodes [s][p] and back
// with no transposition through LDS (the kernel uses none) and no operand
// selects.  Entry layouts: modes (b, a); nodes (s, p); edge values (edge,
// node) with the edges east, west, north, south.
//
//   nodes     mfma(mfma(Q, K), K), K[b][s] = P~_b(x_s)
//   own edges mfma(E, K), E[k][edge]: columns east/west from Q^T and the
//             edge values P~(+-1), columns north/south from Q
//   neighbours the same from the four neighbours' coefficients, one column
//             each (the zero columns of the tables add exact zeros, so both
//             sides of an edge form its traces by the same operations)
//   edges     Rusanov flux, one edge node per lane, on (h, normal momentum,
//             tangential momentum): which of hu and hv is the normal one is
//             settled by which coefficients enter which column
//   back      nodal terms and edge fluxes through the row tables, with the
//             metric factors, 1/R, the weights and the surface signs folded
//             into the tables
//
// What bounds it: the vector pipe.  An FP64 MFMA holds it for 16 cycles and
// the ordinary instructions between them do not overlap with it (measured:
// 18.5 cycles at the nominal clock for the one, 5.3 for an FP64 FMA, 24 for
// the pair), so a group of four elements costs 53 MFMAs and about 160
// instructions, 1650 cycles, against about 1900 for the sum-factorised form
// with its LDS transposes, its operand selects and the fluxes' scaling.  At
// 1440x720 the pipe is busy about three quarters of the time.  Per stage,
// before (sum-factorised half layout) and now: 1440x720 296 -> 265 us, 180x90
// 8.2 -> 7.6, 50x50 RK4 5.2 -> 3.9, 300x300 with 16 layers RK4 477 -> 417.
// The fetch straight into LDS is what makes it pay: with 8-byte gathers in the
// operand layouts the address units were busy 93 % of the time (1440x720 405
// us).  The edges' coefficients formed with FMAs from LDS instead of MFMAs with
// mostly zero columns (35 MFMAs a group) was not faster: five times the bank
// conflicts (285 against 283 us, 180x90 8.0 against 7.6).
#pragma once

#include "dgsw_stage.hpp"

namespace dgsw {

// The cases that run here.
template <typename T, int NP>
constexpr bool M4 = sizeof(T) == 8 && NP == 4;

constexpr int kM4Lds = 1280;  // LDS values per wavefront (M4Lds)

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// 16 bytes a lane, from OFF values behind p, straight into LDS at dst (the
// wavefront's bytes in lane order).
typedef __attribute__((address_space(3))) double lds_double;
template <int OFF = 0>
__device__ __forceinline__ void load_lds16(const double *p, lds_double *dst) {
  typedef const __attribute__((address_space(1))) void gptr;
  typedef __attribute__((address_space(3))) void lptr;
  // the instruction's offset moves both addresses
  __builtin_amdgcn_global_load_lds((gptr *)p, (lptr *)(dst - OFF), 16, OFF * 8, 0);
}

// The tables of the mesh, this lane's entries; kept lane by lane behind the
// mesh's GlobTab (value n of lane l at n 64 + l, m4_lane_tables), so that a
// wavefront reads each with one contiguous load.
struct M4Tab {
  double K;                   // P~_x(xi_y)
  double eX, eY;              // own edges: P~_x(+-1) in columns 0, 1 / 2, 3
  double nE, nW, nN, nS;      // the neighbours' facing edges: column 0 / 1 / 2 / 3
  double DW, BW;              // cF/R w_x P~'_y(xi_x), w_x P~_y(xi_x)
  double PE;                  // -+ cF/(2R) P~_y(+-1) in rows 0, 1 (the flux sums carry the 1/2)
  double sNS;                 // -+ cG/(2R) in rows 2, 3
  double h2;                  // 2 H at mode (0, 0)
  double H, g, alpha, cGR;    // reference depth, gravity, fixed speed, cG/R (wave-uniform)
};
constexpr int kM4Tabs = 12;
constexpr size_t kM4TabOff = (sizeof(GlobTab<double, 4>) + 255) / 256 * 256;   // bytes behind the GlobTab's start
constexpr size_t kM4GlobBytes = kM4TabOff + kM4Tabs * 64 * sizeof(double);

inline void m4_lane_tables(const GlobTab<double, 4> &G, double *dst) {
  const double fx = G.cF * G.invR, fy = G.cG * G.invR;
  for (int l = 0; l < 64; ++l) {
    const int x = l / 16, y = l % 4;
    const double v[kM4Tabs] = {
        G.B[y][x],
        y == 0 ? G.Pp[x] : (y == 1 ? G.Pm[x] : 0.0),
        y == 2 ? G.Pp[x] : (y == 3 ? G.Pm[x] : 0.0),
        y == 0 ? G.Pm[x] : 0.0,
        y == 1 ? G.Pp[x] : 0.0,
        y == 2 ? G.Pm[x] : 0.0,
        y == 3 ? G.Pp[x] : 0.0,
        fx * G.w[x] * G.D[x][y],
        G.w[x] * G.B[x][y],
        x == 0 ? -0.5 * fx * G.Pp[y] : (x == 1 ? 0.5 * fx * G.Pm[y] : 0.0),
        x == 2 ? -0.5 * fy : (x == 3 ? 0.5 * fy : 0.0),
        x == 0 && y == 0 ? G.two_href : 0.0};
    for (int n = 0; n < kM4Tabs; ++n) dst[n * 64 + l] = v[n];
  }
}

__device__ __forceinline__ M4Tab m4_tables(const GlobTab<double, 4> *__restrict__ gt, int lane) {
  const double *__restrict__ p =
      reinterpret_cast<const double *>(reinterpret_cast<const unsigned char *>(gt) + kM4TabOff) + lane;
  M4Tab t;
  t.K = p[0];
  t.eX = p[64];
  t.eY = p[2 * 64];
  t.nE = p[3 * 64];
  t.nW = p[4 * 64];
  t.nN = p[5 * 64];
  t.nS = p[6 * 64];
  t.DW = p[7 * 64];
  t.BW = p[8 * 64];
  t.PE = p[9 * 64];
  t.sNS = p[10 * 64];
  t.h2 = p[11 * 64];
  t.H = gt->href;
  t.g = gt->g;
  t.alpha = gt->alpha;
  t.cGR = gt->cG * gt->invR;
  return t;
}

// A group: up to four consecutive elements from e0 on (below e_end), the first
// in row j0, the others in it or in the next one; off: its layer's offset.
struct M4Group {
  int e0, e_end, j0;
  long long off;
};

// Group k of a layer at offset off.
__device__ __forceinline__ M4Group m4_group(int n_lon, int n_lat, int k, long long off) {
  const bool wide = n_lon >= kM4Elems;
  M4Group g;
  g.e0 = k * (wide ? kM4Elems : n_lon);
  g.j0 = wide ? (unsigned)g.e0 / (unsigned)n_lon : k;
  g.e_end = wide ? n_lon * n_lat : g.e0 + n_lon;
  g.off = off;
  return g;
}

// This lane's element (k: its place in the group; lanes past the last element
// work on a copy of it).
struct M4Elem {
  int e, i, j;
  bool live;
};
__device__ __forceinline__ M4Elem m4_elem(const M4Group &g, int n_lon, int k) {
  M4Elem m;
  m.live = g.e0 + k < g.e_end;
  m.e = m.live ? g.e0 + k : g.e_end - 1;
  m.j = g.j0;
  m.i = m.e - g.j0 * n_lon;
  if (m.i >= n_lon) { m.i -= n_lon; ++m.j; }
  return m;
}

// LDS of one wavefront.  An array [16] of four elements fills 32 chunks of 16
// bytes (64 values); chunk (half, element, row parity, column pair) holds row
// 2 half + parity and columns 2 (pair ^ half) + 0, 1, so that reads in either
// orientation touch every bank once a half wavefront.
struct M4Lds {
  static constexpr int A = 64;                // one array
  static constexpr int Own = 0, N = A;        // variable v at + 2 v A
  static constexpr int Halo = 6 * A, S = 7 * A;
  static constexpr int Q0 = 12 * A;           // q^n, variable v at + v A
  static constexpr int Row = 15 * A;          // the tables of rows j0 and j0 + 1
  static constexpr int Out = 17 * A;          // the results, variable v at + v A
};
static_assert(M4Lds::Out + 3 * M4Lds::A == kM4Lds, "LDS of a wavefront");

// Everything a group reads, fetched straight into LDS 16 bytes a lane (gathers
// of 8 bytes in the operand layouts touch 16 cache lines an instruction: the
// address units then bound the kernel).  The longitude neighbours are the
// group's own elements but for the four of the halo: the one west of the
// first, the one east of the last, and at a row end the first of row j0 and
// the last of row j0 + 1.
__device__ __forceinline__ void m4_fetch(const StageArgs<double, 4> &A, const M4Group &g, bool use_q0, int lane,
                                         lds_double *sh) {
  const int n_lon = A.n_lon, n_lat = A.n_lat, k = (lane >> 2) & 3;
  const M4Elem m = m4_elem(g, n_lon, k);
  // across a pole (no flux there) the element stands in for its neighbour; the
  // zero columns of the edge tables would let a non-finite other one into every
  // trace
  const int eN = m.j < n_lat - 1 ? m.e + n_lon : (A.periodic_y ? m.i : m.e);
  const int eS = m.j > 0 ? m.e - n_lon : (A.periodic_y ? (n_lat - 1) * n_lon + m.i : m.e);
  const int r0 = g.j0 * n_lon, j1 = g.j0 + 1 < n_lat ? g.j0 + 1 : g.j0;
  const int h0 = g.e0 == r0 ? r0 + n_lon - 1 : g.e0 - 1;
  const int h1 = g.e0 + kM4Elems < n_lon * n_lat ? g.e0 + kM4Elems : n_lon * n_lat - 1;
  const int h2 = r0, h3 = (j1 + 1) * n_lon - 1;
  const int eH = k & 2 ? (k & 1 ? h3 : h2) : (k & 1 ? h1 : h0);
  const bool up = lane >= 32;                 // the upper lanes fetch another array than the lower ones
  const int half = (lane >> 4) & 1, rr = 2 * half + ((lane >> 1) & 1), cc = (lane & 1) ^ half;
  const int co = 4 * rr + 2 * cc;
  const double *q = A.q + g.off + co;
  const double *c0 = q + (size_t)(unsigned)(up ? eN : m.e) * 48;
  const double *c1 = q + (size_t)(unsigned)(up ? eS : eH) * 48;
  load_lds16<0>(c0, sh + M4Lds::Own);
  load_lds16<0>(c1, sh + M4Lds::Halo);
  load_lds16<16>(c0, sh + M4Lds::Own + 2 * M4Lds::A);
  load_lds16<16>(c1, sh + M4Lds::Halo + 2 * M4Lds::A);
  load_lds16<32>(c0, sh + M4Lds::Own + 4 * M4Lds::A);
  load_lds16<32>(c1, sh + M4Lds::Halo + 4 * M4Lds::A);
  // q^n; the last array shares its load with row j0's tables (29 chunks)
  const double *c2 = (use_q0 ? A.q0 + g.off + co : q) + (size_t)(unsigned)m.e * 48;
  if (use_q0) load_lds16<0>(c2 + (up ? 16 : 0), sh + M4Lds::Q0);
  const int ch = 2 * ((lane & 31) < 29 ? (lane & 31) : 28);
  const double *rt = reinterpret_cast<const double *>(A.rows + g.j0) + ch;
  load_lds16<0>(up ? rt : c2 + 32, sh + M4Lds::Q0 + 2 * M4Lds::A);
  if (g.e0 + kM4Elems > r0 + n_lon && !up)
    load_lds16<0>(reinterpret_cast<const double *>(A.rows + j1) + ch, sh + M4Lds::Row + M4Lds::A);
}

// What a lane holds of its group: entries (x, y) of every array, or (y, x).
struct M4Data {
  double Q[3], Qt[3], QE[3], QW[3], QN[3], QS[3], qn[3];
  double BM, DM, cs, fc, sn, st, mns, ce;
};

__device__ __forceinline__ int m4_at(int x, int y, int k) {   // value (x, y) of element k's array
  return ((x >> 1) * 16 + k * 4 + 2 * (x & 1) + ((y >> 1) ^ (x >> 1))) * 2 + (y & 1);
}

__device__ __forceinline__ M4Data m4_read(const StageArgs<double, 4> &A, const M4Group &g, bool use_q0, int lane,
                                          const lds_double *sh) {
  using R_ = ShapeH2<double, 4>;              // offsets of the row table's entries
  static_assert(sizeof(RowTab<double, 4>) == 29 * 16 && sizeof(RowTab<double, 4>) == 8 * R_::RP, "row table copy");
  const int x = lane >> 4, y = lane & 3, k = (lane >> 2) & 3, n_lon = A.n_lon;
  const M4Elem m = m4_elem(g, n_lon, k);
  const int pn = m4_at(x, y, k), p0 = m4_at(y, x, 0);
  // the longitude neighbours' places
  const int pE = p0 + (m.i + 1 == n_lon ? M4Lds::Halo + 2 * 8 : (k < 3 ? (k + 1) * 8 : M4Lds::Halo + 8));
  const int pW = p0 + (m.i == 0 && m.j > g.j0 ? M4Lds::Halo + 3 * 8 : (k > 0 ? (k - 1) * 8 : M4Lds::Halo));
  M4Data d;
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    const lds_double *s = sh + 2 * v * M4Lds::A;
    d.Q[v] = s[M4Lds::Own + pn];
    d.Qt[v] = s[M4Lds::Own + p0 + 8 * k];
    d.QE[v] = s[M4Lds::Own + pE];
    d.QW[v] = s[M4Lds::Own + pW];
    d.QN[v] = s[M4Lds::N + pn];
    d.QS[v] = s[M4Lds::S + pn];
    d.qn[v] = use_q0 ? sh[M4Lds::Q0 + v * M4Lds::A + pn] : 0.0;
  }
  const lds_double *rt = sh + M4Lds::Row + M4Lds::A * (m.j - g.j0);
  d.BM = rt[R_::rBM + 4 * x + y];
  d.DM = rt[R_::rDM + 4 * x + y];
  d.cs = rt[R_::rCos + x];
  d.fc = rt[R_::rFc + x];
  d.sn = rt[R_::rSnR + x];
  d.st = rt[R_::rStR + x];
  d.mns = rt[(x == 3 ? R_::rMS : R_::rMN) + y];
  d.ce = rt[x == 3 ? R_::rBot : R_::rTop];
  return d;
}

// The operands read only by the general combination and the forcing.
struct M4More {
  double f[3], a[3], b[3];
};
template <int CM, bool MORE>
__device__ __forceinline__ M4More m4_more(const StageArgs<double, 4> &A, const M4Group &g, int lane) {
  M4More o;
  const M4Elem m = m4_elem(g, A.n_lon, (lane >> 2) & 3);
  const size_t base = g.off + (size_t)m.e * 48 + 4 * (lane >> 4) + (lane & 3);
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    o.f[v] = MORE && A.forcing ? A.forcing[base + 16 * v] : 0.0;
    o.a[v] = MORE && CM == 2 && A.qa ? A.qa[base + 16 * v] : 0.0;
    o.b[v] = MORE && CM == 2 && A.qb ? A.qb[base + 16 * v] : 0.0;
  }
  return o;
}

// The stage from a group's data; polar: some of it lies in a row at a pole.
// Leaves the results in sh (M4Lds::Out).
template <int CM>
__device__ __forceinline__ void m4_compute(const StageArgs<double, 4> &A, const M4Tab &t, M4Data &d, const M4More &o,
                                           const bool polar, const int lane, lds_double *sh) {
  constexpr int combine = CM;
  const int x = lane >> 4, y = lane & 3, k = (lane >> 2) & 3;
  const double H = t.H, grav = t.g;
  const double hq = d.Q[0] - t.h2;
  d.Qt[0] -= t.h2;
  d.QE[0] -= t.h2;
  d.QW[0] -= t.h2;
  d.QN[0] -= t.h2;
  d.QS[0] -= t.h2;

  // ---- nodal values (s, p) = (x, y)
  double nd[3];
  nd[0] = mfma4(hq, t.K, 0.0);
  nd[1] = mfma4(d.Q[1], t.K, 0.0);
  nd[2] = mfma4(d.Q[2], t.K, 0.0);
#pragma unroll
  for (int v = 0; v < 3; ++v) nd[v] = mfma4(nd[v], t.K, 0.0);

  // ---- edge traces (edge, node) = (x, y): h, the normal and the tangential
  // momentum (hu, hv on the longitude edges, hv, hu on the latitude ones)
  double ow[3], nb[3];
  ow[0] = mfma4(hq, t.eY, mfma4(d.Qt[0], t.eX, 0.0));
  ow[1] = mfma4(d.Q[2], t.eY, mfma4(d.Qt[1], t.eX, 0.0));
  ow[2] = mfma4(d.Q[1], t.eY, mfma4(d.Qt[2], t.eX, 0.0));
  nb[0] = mfma4(d.QS[0], t.nS, mfma4(d.QN[0], t.nN, mfma4(d.QW[0], t.nW, mfma4(d.QE[0], t.nE, 0.0))));
  nb[1] = mfma4(d.QS[2], t.nS, mfma4(d.QN[2], t.nN, mfma4(d.QW[1], t.nW, mfma4(d.QE[1], t.nE, 0.0))));
  nb[2] = mfma4(d.QS[1], t.nS, mfma4(d.QN[1], t.nN, mfma4(d.QW[2], t.nW, mfma4(d.QE[2], t.nE, 0.0))));
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    ow[v] = mfma4(ow[v], t.K, 0.0);
    nb[v] = mfma4(nb[v], t.K, 0.0);
  }

  // ---- Rusanov flux, twice the bracket (the 1/2 is in the tables): the own
  // side is the minus side of the east and north edges
  double fl[3];
  {
    const double ho = ow[0] + H, hn = nb[0] + H;
    const double uo = ow[1] * dg_rcp(ho), un = nb[1] * dg_rcp(hn);
    const double po = 0.5 * grav * ow[0] * (ho + H), pn = 0.5 * grav * nb[0] * (hn + H);
    double a;
    if (A.alpha_global != 0) a = t.alpha;
    else a = fmax(fabs(uo) + dg_sqrt(grav * ho), fabs(un) + dg_sqrt(grav * hn));
    if (x & 1) a = -a;
    fl[0] = (ow[1] + nb[1]) - a * (nb[0] - ow[0]);
    fl[1] = ((ow[1] * uo + po) + (nb[1] * un + pn)) - a * (nb[1] - ow[1]);
    fl[2] = (ow[2] * uo + nb[2] * un) - a * (nb[2] - ow[2]);
  }
  // the edge cosine is exactly 0 at a pole edge: no flux, whatever the trace
  // there (a negative depth has none to multiply by 0)
  if (polar) {
    const bool pole = (x & 2) && d.ce == 0.0;
#pragma unroll
    for (int v = 0; v < 3; ++v) fl[v] = pole ? 0.0 : fl[v];
  }

  double res[3] = {o.f[0], o.f[1], o.f[2]};
  // ---- node terms at (s, p): F, G (without cos, in the table) and sources
  const double h = nd[0] + H;
  const double rh = dg_rcp(h);
  const double u = nd[1] * rh, vv = nd[2] * rh;
  const double pr = 0.5 * grav * nd[0] * (h + H);
  const double F1 = nd[1] * u + pr, F2 = nd[1] * vv, G2 = nd[2] * vv + pr;
  const double C = d.fc + u * d.sn;
  const double S1 = C * nd[2], S2 = -(pr * d.st + C * nd[1]);

  // ---- back to modes: contracted over the latitude nodes into (p, b), the
  // latitude edges added; then over the longitude nodes into (b, a), and the
  // longitude edges through (s, a)
  const double GM = d.DM * (d.cs * t.cGR);
  const double EN = t.sNS * (d.ce * d.mns);
  double zf[3], zg[3];
  zf[0] = mfma4(nd[1], d.BM, 0.0);
  zf[1] = mfma4(F1, d.BM, 0.0);
  zf[2] = mfma4(F2, d.BM, 0.0);
  zg[0] = mfma4(nd[2], GM, 0.0);
  zg[1] = mfma4(F2, GM, 0.0);
  zg[2] = mfma4(G2, GM, 0.0);
  zg[1] = mfma4(S1, d.BM, zg[1]);
  zg[2] = mfma4(S2, d.BM, zg[2]);
  zg[0] = mfma4(fl[0], EN, zg[0]);
  zg[1] = mfma4(fl[2], EN, zg[1]);
  zg[2] = mfma4(fl[1], EN, zg[2]);
  double ex[3];
#pragma unroll
  for (int v = 0; v < 3; ++v) ex[v] = mfma4(fl[v], t.PE, 0.0);
#pragma unroll
  for (int v = 0; v < 3; ++v) res[v] = mfma4(zf[v], t.DW, res[v]);
#pragma unroll
  for (int v = 0; v < 3; ++v) res[v] = mfma4(zg[v], t.BW, res[v]);
#pragma unroll
  for (int v = 0; v < 3; ++v) res[v] = mfma4(d.BM, ex[v], res[v]);

  // ---- epilogue
  const int pn = m4_at(x, y, k);
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    double r = res[v];
    if (combine == 2) {
      const double b0 = d.qn[v];
      r = b0 + A.dt * r + (A.c1 * (d.Q[v] - b0) + (A.ca * (o.a[v] - b0) + A.cb * (o.b[v] - b0)));
    } else if (combine) {
      const double yv = d.Q[v] + A.dt * r;
      r = yv + A.c0 * (d.qn[v] - yv) + A.ce * yv;
    }
    sh[M4Lds::Out + v * M4Lds::A + pn] = r;
  }
}

// The results of a group from LDS to memory, 16 bytes a lane.
__device__ __forceinline__ void m4_store(const StageArgs<double, 4> &A, const M4Group &g, int lane, const lds_double *sh) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  const M4Elem m = m4_elem(g, A.n_lon, (lane >> 2) & 3);
  const bool up = lane >= 32;
  const int half = (lane >> 4) & 1, rr = 2 * half + ((lane >> 1) & 1), cc = (lane & 1) ^ half;
  typedef const __attribute__((address_space(3))) d2 lds_d2;
  const d2 o0 = *(lds_d2 *)(sh + M4Lds::Out + 2 * lane);
  const d2 o1 = *(lds_d2 *)(sh + M4Lds::Out + 2 * M4Lds::A + 2 * (lane & 31));
  double *p = A.out + g.off + (size_t)m.e * 48 + 4 * rr + 2 * cc;
  if (m.live) {
    *reinterpret_cast<d2 *>(p + (up ? 16 : 0)) = o0;
    if (!up) *reinterpret_cast<d2 *>(p + 32) = o1;
  }
}

// Waits for everything a group reads to be in LDS (vmcnt(0)); and for this
// lane's reads of it (lgkmcnt(0)), before the next group's arrive.
__device__ __forceinline__ void m4_fetched() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0f70);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void m4_have_read() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);
  asm volatile("" ::: "memory");
}

// `count` groups, group(0) .. group(count - 1), one after the other: the next
// one's data is fetched while the present one is worked on.
template <int CM, bool MORE, typename Group>
__device__ __forceinline__ void m4_run(const StageArgs<double, 4> &A, int count, Group group, int lane,
                                       lds_double *sh) {
  const bool use_q0 = CM == 2 || (CM == 1 && A.c0 != 0.0);
  const M4Tab t = m4_tables(A.gt, lane);
  M4Group g = group(0);
  m4_fetch(A, g, use_q0, lane, sh);
  m4_fetched();
  for (int n = 1;; ++n) {
    M4Data d = m4_read(A, g, use_q0, lane, sh);
    const M4More o = m4_more<CM, MORE>(A, g, lane);
    m4_have_read();
    M4Group next = g;
    if (n < count) {
      next = group(n);
      m4_fetch(A, next, use_q0, lane, sh);
    }
    const int j0 = __builtin_amdgcn_readfirstlane(g.j0);
    const bool polar = !A.periodic_y && (j0 == 0 || j0 + 2 >= A.n_lat);   // (a scalar test: 1 % of a stage saved)
    m4_compute<CM>(A, t, d, o, polar, lane, sh);
    wave_sync();
    // the next group's data before the stores are queued behind them
    if (n < count) m4_fetched();
    m4_store(A, g, lane, sh);
    if (n >= count) break;
    g = next;
  }
}

}  // namespace dgsw
