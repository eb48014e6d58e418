// One whole RK2 substep of the 2D field advance with hyper-resistivity, the
// electron energy equation or open x boundaries, on an LDS tile.  Included by
// the sources of those field advances (one copy per unit).
//
// The stencil-per-stage form (J = curl B, Ohm's law with lap J, Faraday) takes
// six launches a substep, each a pass over arrays that L2 holds: 3 us a launch
// and its host time on small grids, 8 to 10 us at 400 x 800 cells.  Here a
// block takes a tile of 32 x 8 or 32 x 16 cells with a halo of six (each stage
// needs one cell for J, one for lap J and one for curl E) and keeps J, E and
// the stage values in LDS; the overlap with its neighbours is computed again
// (3.4 or 2.4 times the tile's cells at the first step of the first stage,
// none at the last of the second).  The frozen terms are formed in the tile from the
// moments.  51 or 75 KB of LDS: two blocks of 512 threads per CU.
#pragma once

#include "fields_common.hpp"

namespace hvpic {
namespace {

constexpr int kExTX = 32, kExBlock = 512, kExHalo = 6;

template <int HALO, int TY>
struct ExPlane {
  static constexpr int W = kExTX + 2 * HALO, N = W * (TY + 2 * HALO);
  __device__ static int at(int lx, int ly) { return (ly + HALO) * W + lx + HALO; }
};

struct ExtSub {
  // B (B1 when open) as hi + lo and, with the energy equation, the pressure:
  // read from ..in, written to ..out (distinct: a tile reads its neighbours'
  // cells); Lin and PLin null stand for zero
  const float *Bin, *Lin;
  float *Bout, *Lout;
  const float *Pin, *PLin;
  float *Pout, *PLout;
  const float *n, *J;  // the moments held over the subcycle
  const float* B0;     // open: the external field
  float h;
  FGeo g;
  float ilx, ily;      // 1/dx^2, 1/dy^2
  float eta, eta_h, eta_hb;
  int nbuf;
  float gam, kappa0;
  Eos eos;
};

// Hyper-resistivity of column i with the layer of an open box.
__device__ __forceinline__ float tile_eta_h(int i, const ExtSub& A) {
  float e = A.eta_h;
  if (A.nbuf > 0) {
    int d = min(i, A.g.nx - 1 - i);
    d = d > 0 ? d - 1 : 0;
    if (d < A.nbuf) e += A.eta_hb * (1.0f - (float)d / (float)A.nbuf);
  }
  return e;
}

// In an open box a cell's x is its column (a halo cell beyond the ends holds a
// wrapped column, whose values reach no cell of the domain: a ghost column
// takes no x-differences).  The ghost rule of B: the stage value of a ghost
// cell is its interior neighbour's, and the threads of the outermost interior
// cells write the ghosts' new values.
template <bool PE, bool OPEN, int TY>
__global__ __launch_bounds__(kExBlock) void k_ext_sub2d(ExtSub A) {
  using PB = ExPlane<kExHalo, TY>;
  using PJ = ExPlane<kExHalo - 1, TY>;
  using PE1 = ExPlane<kExHalo - 2, TY>;
  using PS = ExPlane<kExHalo - 3, TY>;
  using PP = ExPlane<kExHalo - 4, TY>;  // stage pressure
  __shared__ float sB[3 * PB::N];
  __shared__ float sJ[3 * PJ::N];
  __shared__ float sE[3 * PE1::N];
  __shared__ float sS[3 * PS::N];
  __shared__ float sA[4 * PJ::N];                         // 1/n_f, u_i
  __shared__ float sG[PE ? PJ::N + PP::N : 2 * PE1::N];   // p and p* (PE), or -grad(p_e)/n_f
  const FGeo& g = A.g;
  const int nc = g.ncell, tid = threadIdx.x;
  const int tx0 = blockIdx.x * kExTX, ty0 = blockIdx.y * TY;
  auto gidx = [&](int lx, int ly) {
    int x = tx0 + lx, y = ty0 + ly;
    x %= g.nx; if (x < 0) x += g.nx;
    y %= g.ny; if (y < 0) y += g.ny;
    return x + g.nx * y;
  };
  auto ghost = [&](int lx) { return OPEN && (tx0 + lx == 0 || tx0 + lx == g.nx - 1); };
  // the tile's own cells: one per thread of the first kExTX * TY
  const int ox = tid % kExTX, oy = tid / kExTX;
  const bool own = tid < kExTX * TY && tx0 + ox < g.nx && ty0 + oy < g.ny;
  const int oc = own ? tx0 + ox + g.nx * (ty0 + oy) : 0;
  float lo[3] = {0.f, 0.f, 0.f}, plo = 0.f;
  // every load first, without branches between them
  constexpr int IB = (PB::N + kExBlock - 1) / kExBlock, IJ = (PJ::N + kExBlock - 1) / kExBlock;
  float vb[IB][3], vj[IJ][5];
#pragma unroll
  for (int u = 0; u < IB; ++u) {
    const int t = min(tid + u * kExBlock, PB::N - 1);
    const int c = gidx(t % PB::W - kExHalo, t / PB::W - kExHalo);
#pragma unroll
    for (int a = 0; a < 3; ++a) vb[u][a] = A.Bin[a * nc + c];
  }
#pragma unroll
  for (int u = 0; u < IJ; ++u) {
    const int t = min(tid + u * kExBlock, PJ::N - 1);
    const int c = gidx(t % PJ::W - (kExHalo - 1), t / PJ::W - (kExHalo - 1));
    vj[u][0] = A.n[c];
#pragma unroll
    for (int a = 0; a < 3; ++a) vj[u][1 + a] = A.J[a * nc + c];
    vj[u][4] = PE ? A.Pin[c] : 0.0f;
  }
  if (A.Lin) {
#pragma unroll
    for (int a = 0; a < 3; ++a) lo[a] = A.Lin[a * nc + oc];
    if (PE) plo = A.PLin[oc];
  }
#pragma unroll
  for (int u = 0; u < IB; ++u) {
    const int t = tid + u * kExBlock;
    if (t < PB::N)
#pragma unroll
      for (int a = 0; a < 3; ++a) sB[a * PB::N + t] = vb[u][a];
  }
  float* sP = PE ? sG : sS;  // pressure on PJ: the state, or that of the EOS until B* comes
#pragma unroll
  for (int u = 0; u < IJ; ++u) {
    const int t = tid + u * kExBlock;
    if (t < PJ::N) {
      const float inv = (float)(1.0 / (double)fmaxf(vj[u][0], A.eos.nfloor));
      sA[t] = inv;
#pragma unroll
      for (int a = 0; a < 3; ++a) sA[(1 + a) * PJ::N + t] = vj[u][1 + a] * inv;
      sP[t] = PE ? vj[u][4]
                 : pressure(vj[u][0], A.eos.nfloor, A.eos.te_n0, A.eos.n0, A.eos.gam, A.eos.iso);
    }
  }
  __syncthreads();
  if (!PE) {
    for (int t = tid; t < PE1::N; t += kExBlock) {
      const int ly = t / PE1::W - (kExHalo - 2), lx = t % PE1::W - (kExHalo - 2);
      const int p = PJ::at(lx, ly);
      const float inv = sA[p];
      sG[t] = ghost(lx) ? 0.0f : -(sP[p + 1] - sP[p - 1]) * g.idx2 * inv;
      sG[PE1::N + t] = -(sP[p + PJ::W] - sP[p - PJ::W]) * g.idy2 * inv;
    }
  }
  // J = curl of the planes b (stride W, size N) at slot q
  auto curl = [&](const float* b, int q, int W, int N, bool gh, float* j) {
    const float dyz = (b[2 * N + q + W] - b[2 * N + q - W]) * g.idy2;
    const float dyx = (b[q + W] - b[q - W]) * g.idy2;
    const float dxz = gh ? 0.0f : (b[2 * N + q + 1] - b[2 * N + q - 1]) * g.idx2;
    const float dxy = gh ? 0.0f : (b[N + q + 1] - b[N + q - 1]) * g.idx2;
    j[0] = dyz;
    j[1] = -dxz;
    j[2] = dxy - dyx;
  };
  auto lap = [&](const float* q, int W, bool gh) {
    float r = (q[W] + q[-W] - 2.0f * q[0]) * A.ily;
    if (!gh) r += (q[1] + q[-1] - 2.0f * q[0]) * A.ilx;
    return r;
  };
  // E at (lx, ly) from the stage's B there and J (sJ, on PJ); with the energy
  // equation from the pressure plane p (slot ps, stride pw)
  auto ohm = [&](int lx, int ly, float b0, float b1, float b2, const float* p, int ps, int pw,
                 float* e) {
    const int q = PJ::at(lx, ly), x = tx0 + lx;
    const bool gh = ghost(lx);
    const float inv = sA[q];
    const float j0 = sJ[q], j1 = sJ[PJ::N + q], j2 = sJ[2 * PJ::N + q];
    const float w0 = j0 * inv - sA[PJ::N + q], w1 = j1 * inv - sA[2 * PJ::N + q],
                w2 = j2 * inv - sA[3 * PJ::N + q];
    float g0, g1;
    if (PE) {
      g0 = -(p[ps + 1] - p[ps - 1]) * g.idx2 * inv;
      g1 = -(p[ps + pw] - p[ps - pw]) * g.idy2 * inv;
    } else {
      const int t = PE1::at(lx, ly);
      g0 = sG[t];
      g1 = sG[PE1::N + t];
    }
    const float eh = OPEN ? tile_eta_h(min(max(x, 0), g.nx - 1), A) : A.eta_h;
    float h0 = 0.f, h1 = 0.f, h2 = 0.f;
    if (eh != 0.0f) {
      h0 = eh * lap(sJ + q, PJ::W, gh);
      h1 = eh * lap(sJ + PJ::N + q, PJ::W, gh);
      h2 = eh * lap(sJ + 2 * PJ::N + q, PJ::W, gh);
    }
    e[0] = (w1 * b2 - w2 * b1) + g0 + A.eta * j0 - h0;
    e[1] = (w2 * b0 - w0 * b2) + g1 + A.eta * j1 - h1;
    e[2] = (w0 * b1 - w1 * b0) + 0.0f + A.eta * j2 - h2;
  };
  // dp/dt at (lx, ly) from the pressure plane p (slot ps, stride pw) and J
  auto prate = [&](int lx, int ly, const float* p, int ps, int pw) {
    const int q = PJ::at(lx, ly), W = PJ::W;
    const float* inv = sA;
    const float* ux = sA + PJ::N;
    const float* uy = sA + 2 * PJ::N;
    const float* jx = sJ;
    const float* jy = sJ + PJ::N;
    const float pc = p[ps], pxp = p[ps + 1], pxm = p[ps - 1], pyp = p[ps + pw], pym = p[ps - pw];
    const float uexp = ux[q + 1] - jx[q + 1] * inv[q + 1], uexm = ux[q - 1] - jx[q - 1] * inv[q - 1];
    const float ueyp = uy[q + W] - jy[q + W] * inv[q + W], ueym = uy[q - W] - jy[q - W] * inv[q - W];
    const float uex = ux[q] - jx[q] * inv[q], uey = uy[q] - jy[q] * inv[q];
    const float div = (pxp * uexp - pxm * uexm) * g.idx2 + (pyp * ueyp - pym * ueym) * g.idy2;
    const float adv = uex * (pxp - pxm) * g.idx2 + uey * (pyp - pym) * g.idy2;
    const float tc = pc * inv[q];
    const float lt = (pxp * inv[q + 1] + pxm * inv[q - 1] - 2.0f * tc) * A.ilx +
                     (pyp * inv[q + W] + pym * inv[q - W] - 2.0f * tc) * A.ily;
    const float gm1 = A.gam - 1.0f;
    return -A.gam * div + gm1 * adv + gm1 * A.kappa0 * lt;
  };
  auto b0at = [&](int lx, int ly, float* b) {
    const int c = gidx(lx, ly);
    b[0] += A.B0[c];
    b[1] += A.B0[nc + c];
    b[2] += A.B0[2 * nc + c];
  };
  const float hh = 0.5f * A.h;
  // stage 1: J and E of B
  for (int t = tid; t < PJ::N; t += kExBlock) {
    const int ly = t / PJ::W - (kExHalo - 1), lx = t % PJ::W - (kExHalo - 1);
    float j[3];
    curl(sB, PB::at(lx, ly), PB::W, PB::N, ghost(lx), j);
#pragma unroll
    for (int a = 0; a < 3; ++a) sJ[a * PJ::N + t] = j[a];
  }
  __syncthreads();
  for (int t = tid; t < PE1::N; t += kExBlock) {
    const int ly = t / PE1::W - (kExHalo - 2), lx = t % PE1::W - (kExHalo - 2);
    const int b = PB::at(lx, ly);
    float v[3] = {sB[b], sB[PB::N + b], sB[2 * PB::N + b]}, e[3];
    if (OPEN) b0at(lx, ly, v);
    ohm(lx, ly, v[0], v[1], v[2], sP, PJ::at(lx, ly), PJ::W, e);
#pragma unroll
    for (int a = 0; a < 3; ++a) sE[a * PE1::N + t] = e[a];
  }
  float* sPs = sG + PJ::N;
  if (PE) {
    for (int t = tid; t < PP::N; t += kExBlock) {
      const int ly = t / PP::W - (kExHalo - 4), lx = t % PP::W - (kExHalo - 4);
      const int q = PJ::at(lx, ly);
      sPs[t] = sP[q] + hh * prate(lx, ly, sP, q, PJ::W);
    }
  }
  __syncthreads();
  // B* = B - (h/2) curl E
  for (int t = tid; t < PS::N; t += kExBlock) {
    const int ly = t / PS::W - (kExHalo - 3);
    int lx = t % PS::W - (kExHalo - 3);
    if (OPEN) lx += tx0 + lx == 0 ? 1 : (tx0 + lx == g.nx - 1 ? -1 : 0);
    const int b = PB::at(lx, ly);
    float ce[3];
    curl(sE, PE1::at(lx, ly), PE1::W, PE1::N, false, ce);
#pragma unroll
    for (int a = 0; a < 3; ++a) sS[a * PS::N + t] = sB[a * PB::N + b] - hh * ce[a];
  }
  __syncthreads();
  // stage 2: J (on PP) and E (on a one-cell halo) of B*
  for (int t = tid; t < PP::N; t += kExBlock) {
    const int ly = t / PP::W - (kExHalo - 4), lx = t % PP::W - (kExHalo - 4);
    float j[3];
    curl(sS, PS::at(lx, ly), PS::W, PS::N, ghost(lx), j);
    const int q = PJ::at(lx, ly);
#pragma unroll
    for (int a = 0; a < 3; ++a) sJ[a * PJ::N + q] = j[a];
  }
  __syncthreads();
  {
    constexpr int W = kExTX + 2, N = W * (TY + 2);
    for (int t = tid; t < N; t += kExBlock) {
      const int ly = t / W - 1, lx = t % W - 1;
      const int b = PS::at(lx, ly), q = PE1::at(lx, ly);
      float v[3] = {sS[b], sS[PS::N + b], sS[2 * PS::N + b]}, e[3];
      if (OPEN) b0at(lx, ly, v);
      ohm(lx, ly, v[0], v[1], v[2], sPs, PP::at(lx, ly), PP::W, e);
#pragma unroll
      for (int a = 0; a < 3; ++a) sE[a * PE1::N + q] = e[a];
    }
  }
  __syncthreads();
  if (!own || ghost(ox)) return;
  // B <- B - h curl E (and p), as compensated sums
  const int b = PB::at(ox, oy);
  float ce[3];
  curl(sE, PE1::at(ox, oy), PE1::W, PE1::N, false, ce);
  const bool left = OPEN && tx0 + ox == 1, right = OPEN && tx0 + ox == g.nx - 2;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int q = a * nc + oc;
    const float hi = sB[a * PB::N + b];
    const float y = lo[a] + -A.h * ce[a];
    const float t = hi + y, l = y - (t - hi);
    A.Bout[q] = t;
    A.Lout[q] = l;
    if (left) {
      A.Bout[q - 1] = t;
      A.Lout[q - 1] = l;
    }
    if (right) {
      A.Bout[q + 1] = t;
      A.Lout[q + 1] = l;
    }
  }
  if (PE) {
    const float hi = sP[PJ::at(ox, oy)];
    const float y = plo + A.h * prate(ox, oy, sPs, PP::at(ox, oy), PP::W);
    const float t = hi + y;
    A.PLout[oc] = y - (t - hi);
    A.Pout[oc] = t;
  }
}

// Tiles of 16 rows where those of 8 would not all be resident at once (two
// blocks per CU) and not as many: fewer cells computed twice (402 x 800 cells
// beside the open sort: 45 us a substep with 8 rows, 43 with 16); smaller grids
// spread over more CUs with 8 (256 x 192: 6.1 us).
struct ExtTiles {
  int rows;
  unsigned nx, ny;
};
inline ExtTiles ext_tiles(const FGeo& g) {
  const unsigned nx = (unsigned)ceil_div(g.nx, kExTX);
  const unsigned n8 = (unsigned)ceil_div(g.ny, 8), n16 = (unsigned)ceil_div(g.ny, 16);
  if (nx * n8 > 512 && n8 > n16) return ExtTiles{16, nx, n16};
  return ExtTiles{8, nx, n8};
}

// Whether a grid takes its substeps tile by tile.  A narrow one leaves most of
// each tile empty, and the stencil per stage, which costs six launches and a
// time that goes by the cells, is faster when it has many such tiles (4 x 100000
// cells, four substeps: 135 us against 321).  The line is drawn at the tiles in
// excess of twice those that the cells would fill.  Near it, by tiles / by
// stages: hyper-resistive 8 x 25000 cells (excess 782) 116 / 115 us, 4 x 25000
// (1172) 108 / 94, 8 x 50000 (1563) 186 / 148; open 10 x 12500 (293) 97 / 107,
// 6 x 12500 (485) 96 / 100, 8 x 16666 (522) 115 / 105, 10 x 25000 (587) 148 / 123.
template <bool OPEN>
bool ext_by_tiles(const FGeo& g) {
  const ExtTiles T = ext_tiles(g);
  const int64_t full = (int64_t)g.ncell / (kExTX * T.rows / 2);
  return (int64_t)T.nx * T.ny - full <= (OPEN ? 450 : 1000);
}

template <bool PE, bool OPEN>
void launch_ext_sub2d(hipStream_t s, const ExtSub& A) {
  const ExtTiles T = ext_tiles(A.g);
  if (T.rows == 16)
    hipLaunchKernelGGL((k_ext_sub2d<PE, OPEN, 16>), dim3(T.nx, T.ny), dim3(kExBlock), 0, s, A);
  else
    hipLaunchKernelGGL((k_ext_sub2d<PE, OPEN, 8>), dim3(T.nx, T.ny), dim3(kExBlock), 0, s, A);
}

}  // namespace
}  // namespace hvpic
