// lbmhd_kernels.hip -- gfx950 kernels of the lattice Boltzmann MHD update
// (Flint & Vahala, arXiv:1607.08675): fused pull-stream + moment-space
// collision, equilibrium initialisation, encode/decode, macroscopic fields
// and FP64 diagnostics.
//
// Data layout in HBM (one lattice): 19 planes [plane][y][pitch], x fastest.
// Planes 0..8 = f_0..f_8 (D2Q9), 9..13 = g_x,0..4, 14..18 = g_y,0..4 (D2Q5),
// velocities in the order of Sec. 3.  Every plane stores the deviation from
// the rest state (f_i - w_i, g unchanged): this keeps the low-order bits of
// rho u = sum c_i f_i that a plain f_i would spend on the large w_i.
//
// The step is HBM-bound: 19 loads + 19 stores per site against ~200 FP32
// operations, so the kernel is laid out for bandwidth, not for matrix cores.
// A thread owns V consecutive sites of one row (V = 1 for FP32 storage, V = 2
// for FP16 so that every lane moves 4-byte words); a 256-thread block owns
// 256 V consecutive sites.  All 19 gathers are issued before any arithmetic;
// a plane that streams along x is read with the aligned vector of the
// thread's own sites plus one edge element, the +-1 shifts being served by
// the caches; stores are aligned and non-temporal.  Blocks run in plain row
// order (a remap giving each XCD a contiguous band of tiles measured slower).
#include <math.h>

#include <algorithm>
#include <cmath>
#include <tuple>
#include <type_traits>

#include "lbmhd_impl.h"
#include "lbmhd_step_dev.h"

namespace lbk {
namespace {

// dst(x) = C(pre(x)),  pre_i(x) = src_i(x - c_i) (periodic pull; Sec. 1.2
// streaming written as a gather).  Thread t of block b updates sites
// x0 .. x0 + V - 1 of row y, x0 = (b mod tiles_x) * 256 V + t V, y = b / tiles_x.
// V > 1 requires nx % V == 0.
template <int ST, int V, bool LES, bool NT>
__global__ __launch_bounds__(kStepThreads) void k_step(
    const typename Codec<ST>::T* __restrict__ src, typename Codec<ST>::T* __restrict__ dst,
    Geom geo, Rates rt, int tiles_x) {
  const int x0 = ((int(blockIdx.x) % tiles_x) * kStepThreads + int(threadIdx.x)) * V;
  const int y = int(blockIdx.x) / tiles_x;
  if (x0 >= geo.nx) return;
  const int xl = x0 == 0 ? geo.nx - 1 : x0 - 1;       // source of c_x = +1 planes
  const int xr = x0 + V == geo.nx ? 0 : x0 + V;       // source of c_x = -1 planes
  const int ym = y == 0 ? geo.ny - 1 : y - 1;
  const int yp = y == geo.ny - 1 ? 0 : y + 1;
  // source row of a plane with velocity c_y: y - c_y, indexed by c_y + 1
  const unsigned row[3] = {unsigned(yp) * geo.pitch, unsigned(y) * geo.pitch,
                           unsigned(ym) * geo.pitch};
  float v[kNPop][V];
  gather_row<ST, V>(src, geo.plane, x0, xl, xr, row, v);
  collide_sites<V, LES, ST == kFP16S>(v, rt);
  store_row<ST, V, NT>(dst, geo.plane, row[1] + unsigned(x0), v);
}

// ---------------------------- several steps in place (FP32): saved halos
// A row-walking block of the kernels below reads its own tile and strip and D
// rows and columns around them (D: 3 for three steps, 2 for two).  When src
// and dst are one lattice the blocks around it may already have written those,
// so k_halo_save first copies, for every strip boundary, the D rows on either
// side (rows: [boundary][plane][2 D][pitch]) and, for every tile boundary, the
// D columns (cols: [boundary][ny][plane][8], column x0 - D + j at j), boundary
// b being the lower or left edge of strip or tile b.  A block then takes what
// lies outside its tile from the copies.  Inside, it walks upward and stores
// row r only after the last pass that reads it.
struct Halos {
  const float* rows;
  const float* cols;
  int strips;   // strip boundaries
};

template <typename T, bool INP>
struct Ptrs {
  using Src = const T* __restrict__;
  using Dst = T* __restrict__;
};
template <typename T>
struct Ptrs<T, true> {   // one lattice: its loads and stores alias
  using Src = const T*;
  using Dst = T*;
};
template <typename T, bool INP>
using SrcPtr = typename Ptrs<T, INP>::Src;
template <typename T, bool INP>
using DstPtr = typename Ptrs<T, INP>::Dst;

// The source rows y = r - c_y of one gather of row r, indexed by c_y + 1: the
// element offset in a plane of the lattice where the row lies in the strip
// (bit c_y + 1 of `in`), else its place in the copied rows.
struct HaloRows {
  unsigned in;
  unsigned off[3];
  int row[3];   // rows of the copy before it, for plane 0
  int y[3];
};

template <int D>
__device__ __forceinline__ HaloRows halo_rows(int r, int y0, int h, int strip, int strips,
                                              int pitch) {
  HaloRows o;
  o.in = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int y = r - (c - 1), k = y - y0;
    o.in |= k >= 0 && k < h ? 1u << c : 0u;
    o.y[c] = y;
    o.off[c] = unsigned(y) * pitch;
    const int b = k < 0 ? strip : (strip + 1 == strips ? 0 : strip + 1);
    o.row[c] = b * kNPop * (2 * D) + (k < 0 ? D + k : D + k - h);
  }
  return o;
}

// Element of the copied columns at boundary b, row y, column j of plane 0 (the
// planes follow eight elements apart).
__device__ __forceinline__ unsigned halo_col(int b, int ny, int y, int j) {
  return (unsigned(b) * unsigned(ny) + unsigned(y)) * unsigned(kNPop * 8) + unsigned(j);
}

// pre_q at column x of the tile, as gather_row, of the row in `hr`; lc: the
// local column of wt, tile and next the tile's boundaries.
template <int D>
__device__ __forceinline__ void gather_tile(const float* lat, long long P, const Halos& hs,
                                            const HaloRows& hr, int pitch, int ny, int tile,
                                            int next, int lc, int wt, int x, int xl, int xr,
                                            float (&v)[kNPop][1]) {
  if (hr.in == 7u) {   // all three rows in the strip: nearly every pass
    gather_row<LBMHD_FP32, 1>(lat, P, x, xl, xr, hr.off, v);
  } else {
    // (the empty asm keeps the addresses of these few passes out of the
    // registers of the others)
    long long p = P;
    int step = 2 * D * pitch;
    asm("" : "+s"(p), "+s"(step));
#pragma unroll
    for (int q = 0; q < kNPop; ++q) {
      const int c = kPlaneCy[q] + 1;
      const bool in = hr.in >> c & 1u;
      const float* base =
          in ? lat + q * p : hs.rows + ((long long)hr.row[c] * pitch + (long long)q * step);
      const int xs = kPlaneCx[q] == 0 ? x : (kPlaneCx[q] == 1 ? xl : xr);
      v[q][0] = ld_plane<float>(base, (in ? hr.off[c] : 0u) + unsigned(xs));
    }
  }
  // the elements beyond the tile's edge columns, from the copied columns
  // (a thread may be at both edges of a narrow last tile)
  auto edge = [&](int cx, int b, int j) {
    unsigned o[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) o[c] = halo_col(b, ny, hr.y[c], j);
#pragma unroll
    for (int q = 0; q < kNPop; ++q) {
      const int c = kPlaneCy[q] + 1;
      if (kPlaneCx[q] == cx && (hr.in >> c & 1u))
        v[q][0] = ld_plane<float>(hs.cols, o[c] + unsigned(8 * q));
    }
  };
  if (lc == 0) edge(1, tile, D - 1);
  if (lc + 1 == wt) edge(-1, next, D);
}

// The same at a halo column: local column lc < 0 or >= wt, wrapped to x; b: the
// tile boundary it lies at.
template <int D>
__device__ __forceinline__ void gather_halo(const Halos& hs, const HaloRows& hr, int pitch, int ny,
                                            int b, int lc, int wt, int x, int xl, int xr,
                                            float (&v)[kNPop][1]) {
  unsigned o[3];
#pragma unroll
  for (int c = 0; c < 3; ++c)
    o[c] = halo_col(b, ny, hr.y[c], D + (lc < 0 ? lc : lc - wt));
  if (hr.in == 7u) {
#pragma unroll
    for (int q = 0; q < kNPop; ++q)
      v[q][0] = ld_plane<float>(hs.cols, o[kPlaneCy[q] + 1] + unsigned(8 * q - kPlaneCx[q]));
    return;
  }
  int step = 2 * D * pitch;
  asm("" : "+s"(step));
#pragma unroll
  for (int q = 0; q < kNPop; ++q) {
    const int c = kPlaneCy[q] + 1;
    const int xs = kPlaneCx[q] == 0 ? x : (kPlaneCx[q] == 1 ? xl : xr);
    if (hr.in >> c & 1u)
      v[q][0] = ld_plane<float>(hs.cols, o[c] + unsigned(8 * q - kPlaneCx[q]));
    else
      v[q][0] = ld_plane<float>(hs.rows + ((long long)hr.row[c] * pitch + (long long)q * step),
                                unsigned(xs));
  }
}

// Copies the halos (see above): first the rows, one block a row of a plane,
// then the columns, one block 32 rows at a tile boundary.
__global__ __launch_bounds__(256) void k_halo_save(const float* __restrict__ lat,
                                                   float* __restrict__ rows,
                                                   float* __restrict__ cols, Geom g, int D,
                                                   int strip_h, int strips, int tile_w,
                                                   int col_blocks) {
  const int nrow = strips * kNPop * 2 * D, tid = int(threadIdx.x);
  int b = int(blockIdx.x);
  if (b < nrow) {
    const int k = b % (2 * D), q = (b / (2 * D)) % kNPop, s = b / (2 * D * kNPop);
    int y = (s * strip_h - D + k) % g.ny;
    y = y < 0 ? y + g.ny : y;
    const uint4* a = reinterpret_cast<const uint4*>(lat + q * g.plane + (long long)y * g.pitch);
    uint4* o = reinterpret_cast<uint4*>(rows + (long long)b * g.pitch);
    for (int i = tid; i < g.pitch / 4; i += 256) o[i] = a[i];
    return;
  }
  b -= nrow;
  const int t = b / col_blocks, j = tid & 7, y = (b % col_blocks) * 32 + (tid >> 3);
  int x = (t * tile_w - D + j) % g.nx;
  x = x < 0 ? x + g.nx : x;
  if (y >= g.ny || j >= 2 * D) return;
  const unsigned a = unsigned(y) * unsigned(g.pitch) + unsigned(x), o = halo_col(t, g.ny, y, j);
  float v[kNPop];
#pragma unroll
  for (int q = 0; q < kNPop; ++q) v[q] = ld_plane<float>(lat + q * g.plane, a);
#pragma unroll
  for (int q = 0; q < kNPop; ++q) cols[o + unsigned(8 * q)] = v[q];
}

// ------------------------------------------- two steps in one pass over HBM
// dst = C(S(C(S(src)))) for the closures that read no neighbours (plain and
// Smagorinsky-MHD): temporal blocking.  A block of kT2Threads threads owns a
// tile of W = kT2Threads V columns and a strip of `rows` rows of the output
// and walks the strip upward.  Pass t first updates row r = y0 - 1 + t from
// src (gathered as in k_step) on the tile's columns and on one halo column on
// each side, then updates row r - 1 a second time from those results: its
// pre-collision value of plane q is the first update's post-collision value
// at x - c_q.  The intermediate state never reaches HBM.  Planes that move
// along x are handed to the neighbouring columns through LDS, grouped by c_y:
// a plane with c_y = +1 is read two passes after it is written, c_y = 0 one
// pass after, c_y = -1 in the same pass, hence rings of 4, 3 and 2 row slots,
// which lets one barrier per pass order every write before its reads and
// every read before the slot is written again.  Planes with c_x = 0 stay in
// the thread's registers for the same number of passes.  The intermediate
// values pass through the storage codec, so that the result equals two
// k_step launches bit for bit (the collision spells out its fused
// multiply-adds, so the halo sites' single-site copy of it rounds as the
// paired one does).  HBM bytes per site for two steps: one
// read and one write of the lattice, plus halo re-reads of 2 / rows of the
// rows and 4 / W of the columns.
constexpr int kT2Threads = 256;
// LDS rings: 2 planes x 4 slots + 6 x 3 + 2 x 2 plane-rows
constexpr int kT2SlotsA = 4, kT2SlotsB = 3, kT2SlotsC = 2;
constexpr int kT2Slots = 2 * kT2SlotsA + 6 * kT2SlotsB + 2 * kT2SlotsC;
constexpr int kT2BaseB = 2 * kT2SlotsA, kT2BaseC = kT2BaseB + 6 * kT2SlotsB;
// MID: also store the intermediate state (after the first update) to mid;
// each block writes the rows and columns it owns, so every site once.
// INP: src and dst are one lattice, the halos as k_halo_save left them.
template <int ST, int V, bool LES, bool MID, bool INP, bool NT>
__global__ __launch_bounds__(kT2Threads) void k_step2(
    SrcPtr<typename Codec<ST>::T, INP> src, DstPtr<typename Codec<ST>::T, INP> dst,
    typename Codec<ST>::T* __restrict__ mid, Geom geo, Rates rt, int tiles_x, int rows,
    bool xcd_map, Halos halos) {
  static_assert(!INP || (ST == LBMHD_FP32 && V == 1), "in place: FP32");
  using C = Codec<ST>;
  using T = typename C::T;
  constexpr int W = kT2Threads * V;
  __shared__ T lds[kT2Slots][W + 2];   // LDS column s holds local column s - 1
  const int nx = geo.nx, ny = geo.ny;
  const long long P = geo.plane;
  // blocks go round-robin to the eight XCDs: with xcd_map (a multiple of eight
  // strips launched, the last ones possibly past the lattice) each XCD gets
  // whole strips, so that the halo lines that neighbouring tiles share meet in
  // one L2
  int tile, strip;
  if (xcd_map) {
    const int k = int(blockIdx.x) >> 3;
    strip = (int(blockIdx.x) & 7) + 8 * (k / tiles_x);
    tile = k % tiles_x;
  } else {
    tile = int(blockIdx.x) % tiles_x;
    strip = int(blockIdx.x) / tiles_x;
  }
  const int x0 = tile * W;
  const int y0 = strip * rows;
  if (y0 >= ny) return;
  const int wt = min(W, nx - x0);          // columns of this tile
  const int h = min(rows, ny - y0);        // output rows of this strip
  const int next = tile + 1 == tiles_x ? 0 : tile + 1;
  const int lc = int(threadIdx.x) * V;     // first local column of the thread
  const bool active = lc < wt;
  const int x = x0 + lc;
  const int xl = x == 0 ? nx - 1 : x - 1;
  const int xr = x + V >= nx ? x + V - nx : x + V;
  // threads 0 and 1 also update the halo columns x0 - 1 and x0 + wt (wrapped)
  const bool halo = threadIdx.x < 2;
  const int hx = threadIdx.x == 0 ? (x0 == 0 ? nx - 1 : x0 - 1) : (x0 + wt == nx ? 0 : x0 + wt);
  const int hs = threadIdx.x == 0 ? 0 : wt + 1;
  const int hxl = hx == 0 ? nx - 1 : hx - 1;
  const int hxr = hx == nx - 1 ? 0 : hx + 1;

  // c_x = 0 planes of earlier passes: c_y = 0 from the last pass (zc), c_y = +1
  // from the last two (zu1, zu2)
  float zc[3][V], zu1[3][V], zu2[3][V];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int j = 0; j < V; ++j) zc[k][j] = zu1[k][j] = zu2[k][j] = 0.0f;
  int sA = 0, sB = 0;   // t mod kT2SlotsA, t mod kT2SlotsB
  for (int t = 0; t < h + 2; ++t) {
    const int sC = t & 1;
    // first update of row y0 - 1 + t; c_x = 0 planes kept by c_y (nc: 0, nu: +1, nd: -1)
    float nc[3][V], nu[3][V], nd[3][V];
    unsigned row[3];
    HaloRows hr;
    if (INP)
      hr = halo_rows<2>(y0 - 1 + t, y0, h, strip, halos.strips, geo.pitch);
    else
      t2_rows(y0 - 1 + t, geo, row);
    if (active) {
      float v[kNPop][V];
      if constexpr (INP)
        gather_tile<2>(src, P, halos, hr, geo.pitch, ny, tile, next, lc, wt, x, xl, xr, v);
      else
        gather_row<ST, V>(src, P, x, xl, xr, row, v);
      collide_sites<V, LES, ST == kFP16S>(v, rt);
      if (MID && t >= 1 && t <= h) store_row<ST, V, NT>(mid, P, row[1] + unsigned(x), v);
#pragma unroll
      for (int q = 0; q < kNPop; ++q) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const T e = C::enc(v[q][j]);
          const int g = kT2Group[q], i = kT2Index[q], k = kT2Reg[q];
          if (g == 0)
            lds[sA * 2 + i][lc + j + 1] = e;
          else if (g == 1)
            lds[kT2BaseB + sB * 6 + i][lc + j + 1] = e;
          else if (g == 2)
            lds[kT2BaseC + sC * 2 + i][lc + j + 1] = e;
          else if (kPlaneCy[q] == 0)
            nc[k][j] = C::dec(e);
          else if (kPlaneCy[q] == 1)
            nu[k][j] = C::dec(e);
          else
            nd[k][j] = C::dec(e);
        }
      }
    }
    if (halo) {
      float v[kNPop][1];
      if constexpr (INP)
        gather_halo<2>(halos, hr, geo.pitch, ny, threadIdx.x == 0 ? tile : next,
                           threadIdx.x == 0 ? -1 : wt, wt, hx, hxl, hxr, v);
      else
        gather_row<ST, 1>(src, P, hx, hxl, hxr, row, v);
      collide_sites<1, LES, ST == kFP16S>(v, rt);
#pragma unroll
      for (int q = 0; q < kNPop; ++q) {
        const T e = C::enc(v[q][0]);
        const int g = kT2Group[q], i = kT2Index[q];
        if (g == 0)
          lds[sA * 2 + i][hs] = e;
        else if (g == 1)
          lds[kT2BaseB + sB * 6 + i][hs] = e;
        else if (g == 2)
          lds[kT2BaseC + sC * 2 + i][hs] = e;
      }
    }
    __syncthreads();
    // second update of row y0 - 2 + t (from pass 2 on)
    if (t >= 2 && active) {
      const int sB1 = sB == 0 ? kT2SlotsB - 1 : sB - 1;            // (t - 1) mod slots
      const int sA2 = sA >= 2 ? sA - 2 : sA + kT2SlotsA - 2;       // (t - 2) mod slots
      float v[kNPop][V];
#pragma unroll
      for (int q = 0; q < kNPop; ++q) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const int g = kT2Group[q], i = kT2Index[q], k = kT2Reg[q];
          const int sx = lc + j - kPlaneCx[q] + 1;
          if (g == 0)
            v[q][j] = C::dec(lds[sA2 * 2 + i][sx]);
          else if (g == 1)
            v[q][j] = C::dec(lds[kT2BaseB + sB1 * 6 + i][sx]);
          else if (g == 2)
            v[q][j] = C::dec(lds[kT2BaseC + sC * 2 + i][sx]);
          else if (kPlaneCy[q] == 0)
            v[q][j] = zc[k][j];
          else if (kPlaneCy[q] == 1)
            v[q][j] = zu2[k][j];
          else
            v[q][j] = nd[k][j];
        }
      }
      collide_sites<V, LES, ST == kFP16S>(v, rt);
      store_row<ST, V, NT>(dst, P, unsigned(y0 + t - 2) * geo.pitch + unsigned(x), v);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < V; ++j) {
        zu2[k][j] = zu1[k][j];
        zu1[k][j] = active ? nu[k][j] : 0.0f;
        zc[k][j] = active ? nc[k][j] : 0.0f;
      }
    sA = sA == kT2SlotsA - 1 ? 0 : sA + 1;
    sB = sB == kT2SlotsB - 1 ? 0 : sB + 1;
  }
}

// ----------------------------------------- three steps in one pass (FP32)
// The two-step scheme one level deeper: dst = (C S)^3 src for FP32 storage
// and the closures without neighbour terms.  A block owns a tile of kT3Cols
// columns and a strip of `rows` output rows; pass t takes row y0 - 2 + t
// through the first update (from HBM), row y0 - 3 + t through the second
// (from level 1) and row y0 - 4 + t through the third (from level 2, to
// HBM).  The first update also covers two halo columns on each side and the
// second one on each side; a fifth wave owns those four halo columns, so
// that every thread keeps the values of its own column in registers and no
// wave collides more than three times per pass.  Planes with c_x != 0 cross
// to the neighbouring column through one LDS row per plane and level: the
// consumer reads it right after the barrier that publishes it (two barriers
// per pass, after the first and after the second update), and carries the
// c_y = 0 values one pass and the c_y = +1 values two passes in registers,
// as it does for its own c_x = 0 planes.  So each LDS row is rewritten on
// the next pass and a level is 10 plane-rows.  HBM bytes per site for three
// steps: one read and one write of the lattice, plus halo re-reads of
// 4 / rows of the rows and 8 / kT3Cols of the columns.
// MID: also store the states after the first and the second update to mid1
// and mid2 (each block the rows and columns it owns, so every site once).
// INP: as for k_step2.
template <bool LES, bool MID, bool INP, bool NT>
__global__ __launch_bounds__(kT3Threads) void k_step_t3(SrcPtr<float, INP> src,
                                                        DstPtr<float, INP> dst,
                                                        float* __restrict__ mid1,
                                                        float* __restrict__ mid2, Geom geo,
                                                        Rates rt, int tiles_x, int rows,
                                                        bool xcd_map, Halos hs) {
  __shared__ float l1[kT3Rows][kT3Cols + 4];   // first update: column lc + 2
  __shared__ float l2[kT3Rows][kT3Cols + 2];   // second update: column lc + 1
  const int nx = geo.nx, ny = geo.ny;
  const long long P = geo.plane;
  int tile, strip;
  if (xcd_map) {   // whole strips per XCD, as in k_step2
    const int k = int(blockIdx.x) >> 3;
    strip = (int(blockIdx.x) & 7) + 8 * (k / tiles_x);
    tile = k % tiles_x;
  } else {
    tile = int(blockIdx.x) % tiles_x;
    strip = int(blockIdx.x) / tiles_x;
  }
  const int x0 = tile * kT3Cols, y0 = strip * rows;
  if (y0 >= ny) return;
  const int wt = min(kT3Cols, nx - x0), h = min(rows, ny - y0);
  const int next = tile + 1 == tiles_x ? 0 : tile + 1;
  // the thread's column: its own (threads 0 .. kT3Cols - 1) or a halo column
  // (lanes 0 .. 3 of the fifth wave: x0 - 2, x0 - 1, x0 + wt, x0 + wt + 1)
  const int tid = int(threadIdx.x);
  int lc = tid;
  bool has = tid < wt;
  if (tid >= kT3Cols) {
    const int k = tid - kT3Cols;
    has = k < 4;
    lc = k == 0 ? -2 : (k == 1 ? -1 : (k == 2 ? wt : wt + 1));
  }
  const bool up2 = has && lc >= -1 && lc <= wt;   // takes the second update
  const bool up3 = has && lc >= 0 && lc < wt;     // takes the third update
  // LDS columns read for the second and third updates: lc - c_x + c1 and
  // lc - c_x + c2.  Threads that take no such update read columns 1 .. 3 or
  // 0 .. 2 instead (in bounds, never used), so the reads need no branch.
  const int c1 = up2 ? lc + 2 : 2;
  const int c2 = up3 ? lc + 1 : 1;
  int xc = (x0 + lc) % nx;
  if (xc < 0) xc += nx;
  const int xl = xc == 0 ? nx - 1 : xc - 1;
  const int xr = xc == nx - 1 ? 0 : xc + 1;

  // Inputs of earlier passes, per level, for this thread's column: c_y = 0
  // planes from the last pass, c_y = +1 planes from the last two; z: the
  // c_x = 0 planes (3 per c_y), x: the c_x != 0 ones (6 with c_y = 0, 2 with
  // c_y = +1), already taken from column lc - c_x.
  float z1c[3], z1u1[3], z1u2[3], z2c[3], z2u1[3], z2u2[3];
  float x1c[6], x1u1[2], x1u2[2], x2c[6], x2u1[2], x2u2[2];
#pragma unroll
  for (int k = 0; k < 3; ++k) z1c[k] = z1u1[k] = z1u2[k] = z2c[k] = z2u1[k] = z2u2[k] = 0.0f;
#pragma unroll
  for (int k = 0; k < 6; ++k) x1c[k] = x2c[k] = 0.0f;
#pragma unroll
  for (int k = 0; k < 2; ++k) x1u1[k] = x1u2[k] = x2u1[k] = x2u2[k] = 0.0f;
  for (int t = 0; t < h + 4; ++t) {
    // first update of row y0 - 2 + t
    float n1c[3], n1u[3], n1d[3];
    if (has) {
      unsigned row[3];
      float v[kNPop][1];
      if constexpr (INP) {
        const HaloRows hr = halo_rows<3>(y0 - 2 + t, y0, h, strip, hs.strips, geo.pitch);
        if (tid < kT3Cols)
          gather_tile<3>(src, P, hs, hr, geo.pitch, ny, tile, next, lc, wt, xc, xl, xr,
                                        v);
        else
          gather_halo<3>(hs, hr, geo.pitch, ny, lc < 0 ? tile : next, lc, wt, xc, xl, xr,
                                     v);
      } else {
        t2_rows(y0 - 2 + t, geo, row);
        gather_row<LBMHD_FP32, 1>(src, P, xc, xl, xr, row, v);
      }
      collide_sites<1, LES>(v, rt);
      if (MID && up3 && t >= 2 && t <= h + 1)
        store_row<LBMHD_FP32, 1, NT>(mid1, P, row[1] + unsigned(xc), v);
#pragma unroll
      for (int q = 0; q < kNPop; ++q) {
        const int k = kT2Reg[q];
        if (kT2Group[q] >= 0)
          l1[t3_row(q)][lc + 2] = v[q][0];
        else if (kPlaneCy[q] == 0)
          n1c[k] = v[q][0];
        else if (kPlaneCy[q] == 1)
          n1u[k] = v[q][0];
        else
          n1d[k] = v[q][0];
      }
    }
    __syncthreads();
    // second update of row y0 - 3 + t (from pass 2 on); the level-1 row of
    // this pass is read in every pass, before the next one overwrites it
    float n2c[3], n2u[3], n2d[3];
    const bool do2 = t >= 2 && up2;
    {
      float e[kT3Rows];
#pragma unroll
      for (int q = 0; q < kNPop; ++q)
        if (kT2Group[q] >= 0) e[t3_row(q)] = l1[t3_row(q)][c1 - kPlaneCx[q]];
      float v[kNPop][1];
#pragma unroll
      for (int q = 0; q < kNPop; ++q) {
        const int g = kT2Group[q], i = kT2Index[q], k = kT2Reg[q];
        if (g >= 0)
          v[q][0] = g == 0 ? x1u2[i] : (g == 1 ? x1c[i] : e[t3_row(q)]);
        else
          v[q][0] = kPlaneCy[q] == 0 ? z1c[k] : (kPlaneCy[q] == 1 ? z1u2[k] : n1d[k]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x1u2[i] = x1u1[i];
        x1u1[i] = e[i];
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) x1c[i] = e[2 + i];
      if (do2) {
        collide_sites<1, LES>(v, rt);
        if (MID && up3 && t >= 3 && t <= h + 2)
          store_row<LBMHD_FP32, 1, NT>(mid2, P, unsigned(y0 - 3 + t) * geo.pitch + unsigned(xc), v);
#pragma unroll
        for (int q = 0; q < kNPop; ++q) {
          const int k = kT2Reg[q];
          if (kT2Group[q] >= 0)
            l2[t3_row(q)][lc + 1] = v[q][0];
          else if (kPlaneCy[q] == 0)
            n2c[k] = v[q][0];
          else if (kPlaneCy[q] == 1)
            n2u[k] = v[q][0];
          else
            n2d[k] = v[q][0];
        }
      }
    }
    __syncthreads();
    // third update of row y0 - 4 + t (from pass 4 on), stored; the level-2
    // row of this pass is read in every pass, as above
    {
      float e[kT3Rows];
#pragma unroll
      for (int q = 0; q < kNPop; ++q)
        if (kT2Group[q] >= 0) e[t3_row(q)] = l2[t3_row(q)][c2 - kPlaneCx[q]];
      if (t >= 4 && up3) {
        float v[kNPop][1];
#pragma unroll
        for (int q = 0; q < kNPop; ++q) {
          const int g = kT2Group[q], i = kT2Index[q], k = kT2Reg[q];
          if (g >= 0)
            v[q][0] = g == 0 ? x2u2[i] : (g == 1 ? x2c[i] : e[t3_row(q)]);
          else
            v[q][0] = kPlaneCy[q] == 0 ? z2c[k] : (kPlaneCy[q] == 1 ? z2u2[k] : n2d[k]);
        }
        collide_sites<1, LES>(v, rt);
        store_row<LBMHD_FP32, 1, NT>(dst, P, unsigned(y0 - 4 + t) * geo.pitch + unsigned(xc), v);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x2u2[i] = x2u1[i];
        x2u1[i] = e[i];
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) x2c[i] = e[2 + i];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      z1u2[k] = z1u1[k];
      z1u1[k] = has ? n1u[k] : 0.0f;
      z1c[k] = has ? n1c[k] : 0.0f;
      z2u2[k] = z2u1[k];
      z2u1[k] = do2 ? n2u[k] : 0.0f;
      z2c[k] = do2 ? n2c[k] : 0.0f;
    }
  }
}

// --------------------------------------------- steps with lattice gradients
// Same update as k_step for the closures that need the neighbours: the
// kinetic closure (KIN) relaxes toward the filtered equilibria, whose Delta^2
// parts need gradients of rho, j, B; the cross-helicity closure (EDDY = 2)
// needs the vorticity.  The gradients are those of the pre-collision
// (gathered) neighbours, by the isotropic D2Q9 difference
// d_a X = 3 sum_i w_i c_ia X(x + c_i).  A block of kKinThreads threads owns
// as many columns and a strip of kKinRows rows.  It walks the strip row by
// row: it gathers row y+1 (each population is read once), writes that row's
// rho - 1, j (and B for KIN) into a rolling 3-row LDS buffer with one halo
// column on each side, and then collides row y, whose populations it
// gathered on the previous pass.
#ifndef LBMHD_KIN_ROWS
#define LBMHD_KIN_ROWS 16
#endif
#ifndef LBMHD_KIN_THREADS
#define LBMHD_KIN_THREADS 512
#endif
constexpr int kKinRows = LBMHD_KIN_ROWS;
constexpr int kKinThreads = LBMHD_KIN_THREADS;
constexpr int kKinCols = kKinThreads + 2;

// Encoded populations of the pre-collision state at (x, y): pre_q(x) =
// src_q(x - c_q), periodic.  The loads are only issued here; decoding happens
// where the values are used, so they can stay in flight meanwhile.
template <int ST>
__device__ __forceinline__ void load_site(const typename Codec<ST>::T* __restrict__ src,
                                          const Geom& geo, int x, int y,
                                          typename Codec<ST>::T (&p)[kNPop]) {
  const int xm = x == 0 ? geo.nx - 1 : x - 1;
  const int xp = x == geo.nx - 1 ? 0 : x + 1;
  const int ym = y == 0 ? geo.ny - 1 : y - 1;
  const int yp = y == geo.ny - 1 ? 0 : y + 1;
  const unsigned row[3] = {unsigned(yp) * geo.pitch, unsigned(y) * geo.pitch,
                           unsigned(ym) * geo.pitch};
  const long long P = geo.plane;
#pragma unroll
  for (int q = 0; q < kNPop; ++q) {
    const int xs = kPlaneCx[q] == 0 ? x : (kPlaneCx[q] == 1 ? xm : xp);
    p[q] = ld_plane<typename Codec<ST>::T>(src + q * P, row[kPlaneCy[q] + 1] + unsigned(xs));
  }
}

// rho - 1, j_x, j_y, B_x, B_y of gathered populations (deviation variables).
__device__ __forceinline__ void site_moments(const float (&p)[kNPop], float (&m)[5]) {
  m[0] = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])) + p[8];
  m[1] = (p[1] - p[3]) + (p[5] - p[7]) - (p[6] - p[8]);
  m[2] = (p[2] - p[4]) + (p[5] - p[7]) + (p[6] - p[8]);
  m[3] = (p[9] + p[10]) + (p[11] + p[12]) + p[13];
  m[4] = (p[14] + p[15]) + (p[16] + p[17]) + p[18];
}

// Terms of the closures with lattice gradients at one site, from the
// pre-collision rho - 1, j (and B for KIN) of the site and its eight
// neighbours: rows rm (y - 1), r0 (y) and rp (y + 1) of a moment buffer whose
// fields lie `fs` floats apart, the site at column c.  Isotropic D2Q9
// gradient: d_x = (E - W)/3 + (NE - NW + SE - SW)/12, d_y likewise.
// h_X = grad X - X grad(rho) / rho (= rho grad(X / rho)); ratio terms
// (X Y / rho) of the kinetic closure use it, product terms (B B) the plain
// gradients:
//   R(X, Y) = Delta^2 / (12 rho) h_X . h_Y,  S(X, Y) = Delta^2 / 12 grad X . grad Y;
// the vorticity is d_x u_y - d_y u_x = (h_jy,x - h_jx,y) / rho.  Every
// multiply-add is written out (no other contraction), so each kernel that
// evaluates the terms rounds them identically.
template <int EDDY, bool KIN>
__device__ __forceinline__ NbTerms nb_terms(const float* __restrict__ rm,
                                            const float* __restrict__ r0,
                                            const float* __restrict__ rp, int fs, int c,
                                            float c12) {
#pragma clang fp contract(off)
  constexpr int NF = KIN ? 5 : 3;
  float gx[NF], gy[NF], v[NF];
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    const int o = k * fs + c;
    const float e = r0[o + 1], w = r0[o - 1];
    const float nn = rp[o], ss = rm[o];
    const float ne = rp[o + 1], nw = rp[o - 1];
    const float se = rm[o + 1], sw = rm[o - 1];
    gx[k] = fmaf(1.0f / 3.0f, e - w, (1.0f / 12.0f) * ((ne - nw) + (se - sw)));
    gy[k] = fmaf(1.0f / 3.0f, nn - ss, (1.0f / 12.0f) * ((ne + nw) - (se + sw)));
    v[k] = r0[o];
  }
  const float ir = frcp(1.0f + v[0]);
  const float grx = gx[0] * ir, gry = gy[0] * ir;
  float hx[NF - 1], hy[NF - 1];
#pragma unroll
  for (int k = 0; k < NF - 1; ++k) {
    hx[k] = fmaf(-v[k + 1], grx, gx[k + 1]);
    hy[k] = fmaf(-v[k + 1], gry, gy[k + 1]);
  }
  NbTerms kc{0.f, 0.f, 0.f, 0.f, 0.f};
  if constexpr (KIN) {
    const float cr = c12 * ir;
    const float jxjx = cr * fmaf(hx[0], hx[0], hy[0] * hy[0]);
    const float jyjy = cr * fmaf(hx[1], hx[1], hy[1] * hy[1]);
    kc.m3 = fmaf(cr, fmaf(hx[0], hx[1], hy[0] * hy[1]), -(c12 * fmaf(gx[3], gx[4], gy[3] * gy[4])));
    kc.m4 = fmaf(-c12, fmaf(gx[3], gx[3], gy[3] * gy[3]) - fmaf(gx[4], gx[4], gy[4] * gy[4]),
                 jxjx - jyjy);
    kc.m78 = -3.0f * (jxjx + jyjy);
    kc.e = cr * (fmaf(hx[0], hx[3], hy[0] * hy[3]) - fmaf(hx[1], hx[2], hy[1] * hy[2]));
  }
  if constexpr (EDDY == 2) kc.w = (hx[1] - hy[0]) * ir;
  return kc;
}

template <int ST, int EDDY, bool KIN>
__global__ __launch_bounds__(kKinThreads) void k_step_nb(
    const typename Codec<ST>::T* __restrict__ src, typename Codec<ST>::T* __restrict__ dst,
    Geom geo, Rates rt, float c12, int tiles_x) {
  using C = Codec<ST>;
  using T = typename C::T;
  constexpr int NF = KIN ? 5 : 3;   // staged fields: rho - 1, j (, B)
  __shared__ float mac[3][NF][kKinCols];
  const int tx = int(threadIdx.x);
  const int xt = (int(blockIdx.x) % tiles_x) * kKinThreads;
  const int y0 = (int(blockIdx.x) / tiles_x) * kKinRows;
  const int y1 = min(y0 + kKinRows, geo.ny);
  const int x = xt + tx;
  const bool active = x < geo.nx;
  const int xc = x % geo.nx;                                   // column staged by this thread
  const int xh = tx == 0 ? (xt == 0 ? geo.nx - 1 : xt - 1)     // halo column (threads 0, 1)
                         : (xt + kKinThreads) % geo.nx;
  const int ch = tx == 0 ? 0 : kKinCols - 1;
  // Rows are loaded one pass ahead of their use: the loads of row y + 2 (and,
  // in threads 0 and 1, of a halo column) are issued before row y collides,
  // and row y + 1, loaded on the previous pass, is decoded and its moments
  // written to LDS slot `slot` (rows wrap periodically).
  T raw[kNPop], rawh[kNPop];
  auto issue = [&](int yy) {
    yy = yy < 0 ? yy + geo.ny : (yy >= geo.ny ? yy - geo.ny : yy);
    load_site<ST>(src, geo, xc, yy, raw);
    if (tx < 2) load_site<ST>(src, geo, xh, yy, rawh);
  };
  auto commit = [&](int slot, float (&p)[kNPop]) {
#pragma unroll
    for (int q = 0; q < kNPop; ++q) p[q] = C::dec(raw[q]);
    float m[5];
    site_moments(p, m);
#pragma unroll
    for (int k = 0; k < NF; ++k) mac[slot][k][tx + 1] = m[k];
    if (tx < 2) {
      float ph[kNPop], mh[5];
#pragma unroll
      for (int q = 0; q < kNPop; ++q) ph[q] = C::dec(rawh[q]);
      site_moments(ph, mh);
#pragma unroll
      for (int k = 0; k < NF; ++k) mac[slot][k][ch] = mh[k];
    }
  };
  float cur[kNPop], nxt[kNPop];
  issue(y0 - 1);                                  // row y0 - 1: moments only
  commit(0, nxt);
  issue(y0);
  commit(1, cur);
  issue(y0 + 1);
  const long long P = geo.plane;
  for (int y = y0; y < y1; ++y) {
    const int sm = (y - y0) % 3, s0 = (y - y0 + 1) % 3, sp = (y - y0 + 2) % 3;
    commit(sp, nxt);
    if (y + 2 <= y1) issue(y + 2);
    __syncthreads();
    if (active) {
      const NbTerms kc =
          nb_terms<EDDY, KIN>(&mac[sm][0][0], &mac[s0][0][0], &mac[sp][0][0], kKinCols, tx + 1, c12);
      float f[9], g[10];
#pragma unroll
      for (int i = 0; i < 9; ++i) f[i] = cur[i];
#pragma unroll
      for (int k = 0; k < 10; ++k) g[k] = cur[9 + k];
      collide<EDDY, KIN>(f, g, rt, kc);
      const unsigned od = unsigned(y) * geo.pitch + unsigned(x);
#pragma unroll
      for (int i = 0; i < 9; ++i) st_plane_nt<T>(dst + i * P, od, C::enc(f[i]));
#pragma unroll
      for (int k = 0; k < 10; ++k) st_plane_nt<T>(dst + (9 + k) * P, od, C::enc(g[k]));
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kNPop; ++q) cur[q] = nxt[q];
  }
}

// ------------------------ two steps per pass with lattice gradients
// dst = (C S)^2 src for the closures that need the neighbours' moments
// (kinetic, cross-helicity).  The second update at a site needs the first
// update's output two sites out (its own gather reaches one site, the
// gradients of the gathered moments one more), and the first update needs the
// input three sites out for its moments and four for their gathers.  A block
// owns a tile of kNb2Cols columns and a strip of `rows` output rows and walks
// upward; pass t, with a = y0 - 3 + t:
//   1. gathers row a from HBM (columns x0 - 3 .. x0 + wt + 2) and writes its
//      moments to ring m1 (3 rows);
//   2. first update of row a - 1 (columns x0 - 2 .. x0 + wt + 1), with the
//      gradients of rows a - 2 .. a of m1; the planes moving along x go to the
//      neighbouring columns through one LDS row per plane (y1), the others
//      stay in the thread's registers;
//   3. second gather of row a - 2 (columns x0 - 1 .. x0 + wt): each thread
//      reads the y1 values it needs right after the barrier that publishes
//      them and carries them on in registers (c_y = 0 planes one pass, c_y = +1
//      two), as the three-step kernel does; their moments go to ring m2;
//   4. second update of row a - 3 (the tile's own columns), with the
//      gradients of rows a - 4 .. a - 2 of m2, stored.
// Three barriers per pass, between the stages.  A fifth wave owns the six
// halo columns.  The first update's output passes through the storage codec,
// so the result equals two k_step_nb launches bit for bit.  MID: also store
// the intermediate state (each block the rows and columns it owns).  HBM
// bytes per site for two steps: one read and one write of the lattice, plus
// halo re-reads of 6 / rows of the rows and 6 / kNb2Cols of the columns.
constexpr int kNb2Cols = 256;
constexpr int kNb2Threads = kNb2Cols + 64;

// Compiled for at least four waves per SIMD (at most 128 VGPRs): with the
// compiler's own choice the pass measured 1.2x slower for the kinetic and the
// cross-helicity closure and 1.5x slower for both together (135 VGPRs), at
// 4096^2, with bit-identical results.
template <int ST, int EDDY, bool KIN, bool MID, bool NT>
__global__ __launch_bounds__(kNb2Threads) __attribute__((amdgpu_waves_per_eu(4))) void k_step_nb2(
    const typename Codec<ST>::T* __restrict__ src, typename Codec<ST>::T* __restrict__ dst,
    typename Codec<ST>::T* __restrict__ mid, Geom geo, Rates rt, float c12, int tiles_x,
    int rows, bool xcd_map) {
  using C = Codec<ST>;
  using T = typename C::T;
  constexpr int NF = KIN ? 5 : 3;        // staged fields: rho - 1, j (, B)
  constexpr int W = kNb2Cols;
  __shared__ float m1[3][NF][W + 6];     // LDS column lc + 3
  __shared__ T y1[kT3Rows][W + 4];       // LDS column lc + 2
  __shared__ float m2[3][NF][W + 2];     // LDS column lc + 1
  const int nx = geo.nx, ny = geo.ny;
  const long long P = geo.plane;
  int tile, strip;
  if (xcd_map) {   // whole strips per XCD, as in k_step2
    const int k = int(blockIdx.x) >> 3;
    strip = (int(blockIdx.x) & 7) + 8 * (k / tiles_x);
    tile = k % tiles_x;
  } else {
    tile = int(blockIdx.x) % tiles_x;
    strip = int(blockIdx.x) / tiles_x;
  }
  // Kinetic closure with FP32 states: the next pass's first gather is issued
  // right after this pass's first barrier and flies during stages 2 to 4
  // (66.5k against 62.4k MLUPS at 4096^2, 62.8k against 57.9k with les = 3,
  // same results); the cross-helicity closure's registers spill with it
  // (29.7k against 54.6k).
  constexpr bool kPf = ST == LBMHD_FP32 && EDDY != 2;
  const int x0 = tile * W, y0 = strip * rows;
  // a strip past the lattice; the FP16 kinetic pass returns below, as fast as
  // without the test (64^2 15.8 us per step, 17.0 from here; FP32 cross-helicity
  // 4096^2 315.5 from here, 317.5 from below)
  constexpr bool kLate = ST != LBMHD_FP32 && EDDY == 0;
  if (!kLate && y0 >= ny) return;
  const int wt = min(W, nx - x0), h = min(rows, ny - y0);
  // the thread's column: its own (threads 0 .. W - 1) or a halo column
  // (lanes 0 .. 5 of the fifth wave: x0 - 3 .. x0 - 1, x0 + wt .. x0 + wt + 2)
  const int tid = int(threadIdx.x);
  int lc = tid;
  bool has = tid < wt;
  if (tid >= W) {
    const int k = tid - W;
    has = k < 6;
    lc = k < 3 ? k - 3 : wt + (k - 3);
  }
  const bool up2 = has && lc >= -2 && lc <= wt + 1;   // takes the first update
  const bool up3 = has && lc >= -1 && lc <= wt;       // takes the second gather
  const bool up4 = has && lc >= 0 && lc < wt;         // takes the second update
  // y1 column read for the second gather: lc + 2 - c_x (a fixed in-bounds
  // column for the threads that take no second gather)
  const int c3 = up3 ? lc + 2 : 2;
  int xc = (x0 + lc) % nx;
  if (xc < 0) xc += nx;
  const int xl = xc == 0 ? nx - 1 : xc - 1;
  const int xr = xc == nx - 1 ? 0 : xc + 1;

  float p1c[kNPop], p2c[kNPop];        // gathers of the previous pass (rows a - 1, a - 3)
  float z1c[3], z1u1[3], z1u2[3];      // y1, planes with c_x = 0, by c_y and pass
  float x1c[6], x1u1[2], x1u2[2];      // y1, planes with c_x != 0, taken from lc - c_x
#pragma unroll
  for (int q = 0; q < kNPop; ++q) p1c[q] = p2c[q] = 0.0f;
#pragma unroll
  for (int k = 0; k < 3; ++k) z1c[k] = z1u1[k] = z1u2[k] = 0.0f;
#pragma unroll
  for (int k = 0; k < 6; ++k) x1c[k] = 0.0f;
#pragma unroll
  for (int k = 0; k < 2; ++k) x1u1[k] = x1u2[k] = 0.0f;
  float pf[kNPop][1];
  // rows y0 - 3 .. y0 + h + 2: more than one period on a lattice two rows high
  auto gather_at = [&](int r, float (&v)[kNPop][1]) {
    int a = r % ny;
    if (a < 0) a += ny;
    unsigned row[3];
    t2_rows(a, geo, row);
    gather_row<ST, 1>(src, P, xc, xl, xr, row, v);
  };
  if (kLate && h <= 0) return;
  if (kPf && has) gather_at(y0 - 3, pf);
  for (int t = 0; t < h + 6; ++t) {
    const int s0 = t % 3;                         // ring slot of this pass
    const int s1 = s0 == 0 ? 2 : s0 - 1;          // (t - 1) mod 3
    const int s2 = s1 == 0 ? 2 : s1 - 1;          // (t - 2) mod 3
    // 1. gather row a = y0 - 3 + t and stage its moments
    float p1n[kNPop];
    if (has) {
      float v[kNPop][1];
      if (kPf) {
#pragma unroll
        for (int q = 0; q < kNPop; ++q) v[q][0] = pf[q][0];
      } else {
        gather_at(y0 - 3 + t, v);
      }
#pragma unroll
      for (int q = 0; q < kNPop; ++q) p1n[q] = v[q][0];
      float m[5];
      site_moments(p1n, m);
#pragma unroll
      for (int k = 0; k < NF; ++k) m1[s0][k][lc + 3] = m[k];
    }
    __syncthreads();
    if (kPf && has && t + 1 < h + 6) gather_at(y0 - 2 + t, pf);
    // 2. first update of row a - 1 (from pass 2 on)
    float n2c[3], n2u[3], n2d[3];
    const bool do2 = up2 && t >= 2;
    if (do2) {
      const NbTerms kc =
          nb_terms<EDDY, KIN>(&m1[s2][0][0], &m1[s1][0][0], &m1[s0][0][0], W + 6, lc + 3, c12);
      float f[9], g[10];
#pragma unroll
      for (int i = 0; i < 9; ++i) f[i] = p1c[i];
#pragma unroll
      for (int k = 0; k < 10; ++k) g[k] = p1c[9 + k];
      collide<EDDY, KIN>(f, g, rt, kc);
      float v[kNPop];
#pragma unroll
      for (int i = 0; i < 9; ++i) v[i] = f[i];
#pragma unroll
      for (int k = 0; k < 10; ++k) v[9 + k] = g[k];
      const int r1 = y0 - 4 + t;                  // row a - 1
      if (MID && lc >= 0 && lc < wt && r1 >= y0 && r1 < y0 + h) {
        const unsigned od = unsigned(r1) * geo.pitch + unsigned(xc);
#pragma unroll
        for (int q = 0; q < kNPop; ++q) st_plane_as<NT, T>(mid + q * P, od, C::enc(v[q]));
      }
#pragma unroll
      for (int q = 0; q < kNPop; ++q) {
        const T e = C::enc(v[q]);
        const int k = kT2Reg[q];
        if (kT2Group[q] >= 0)
          y1[t3_row(q)][lc + 2] = e;
        else if (kPlaneCy[q] == 0)
          n2c[k] = C::dec(e);
        else if (kPlaneCy[q] == 1)
          n2u[k] = C::dec(e);
        else
          n2d[k] = C::dec(e);
      }
    }
    __syncthreads();
    // 3. second gather of row a - 2 (from pass 4 on); the y1 row of this pass
    // is read in every pass, before the next one overwrites it
    float p2n[kNPop];
    const bool do3 = up3 && t >= 4;
    {
      float e[kT3Rows];
#pragma unroll
      for (int q = 0; q < kNPop; ++q)
        if (kT2Group[q] >= 0) e[t3_row(q)] = C::dec(y1[t3_row(q)][c3 - kPlaneCx[q]]);
#pragma unroll
      for (int q = 0; q < kNPop; ++q) {
        const int g = kT2Group[q], i = kT2Index[q], k = kT2Reg[q];
        if (g >= 0)
          p2n[q] = g == 0 ? x1u2[i] : (g == 1 ? x1c[i] : e[t3_row(q)]);
        else
          p2n[q] = kPlaneCy[q] == 0 ? z1c[k] : (kPlaneCy[q] == 1 ? z1u2[k] : n2d[k]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x1u2[i] = x1u1[i];
        x1u1[i] = e[i];
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) x1c[i] = e[2 + i];
      if (do3) {
        float m[5];
        site_moments(p2n, m);
#pragma unroll
        for (int k = 0; k < NF; ++k) m2[s0][k][lc + 1] = m[k];
      }
    }
    __syncthreads();
    // 4. second update of row a - 3 (from pass 6 on), stored
    if (up4 && t >= 6) {
      const NbTerms kc =
          nb_terms<EDDY, KIN>(&m2[s2][0][0], &m2[s1][0][0], &m2[s0][0][0], W + 2, lc + 1, c12);
      float f[9], g[10];
#pragma unroll
      for (int i = 0; i < 9; ++i) f[i] = p2c[i];
#pragma unroll
      for (int k = 0; k < 10; ++k) g[k] = p2c[9 + k];
      collide<EDDY, KIN>(f, g, rt, kc);
      const unsigned od = unsigned(y0 - 6 + t) * geo.pitch + unsigned(xc);
#pragma unroll
      for (int i = 0; i < 9; ++i) st_plane_as<NT, T>(dst + i * P, od, C::enc(f[i]));
#pragma unroll
      for (int k = 0; k < 10; ++k) st_plane_as<NT, T>(dst + (9 + k) * P, od, C::enc(g[k]));
    }
#pragma unroll
    for (int q = 0; q < kNPop; ++q) {
      p1c[q] = has ? p1n[q] : 0.0f;
      p2c[q] = do3 ? p2n[q] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      z1u2[k] = z1u1[k];
      z1u1[k] = do2 ? n2u[k] : 0.0f;
      z1c[k] = do2 ? n2c[k] : 0.0f;
    }
  }
}

// ------------------------------------------ several steps of a tile in LDS
// dst = (C S)^k src, k >= 1 a run-time argument or K: a block owns a tile of
// the output and a region of RX x RY sites around it, takes the first update of
// every site of the region from HBM (periodic images where the region passes
// the lattice's edge or is larger than the lattice), and the other k - 1 from
// LDS, on a region that shrinks by one site on each side per step.  A thread
// owns the S sites (rx, ry + j RY / S).  It holds
// the rest populations in registers; the 16 moving ones pass through one LDS
// buffer (written, barrier, read at x - c, barrier), in PH parts.  Bound by the
// issue of vector instructions, with the lanes whose sites are halo counted (1.4
// to 1.8 a site and step): at 0.60-0.70 of their nominal issue rate with FP32
// storage (1024^2, 4096^2), 0.87-1.02 with FP16 (8192^2), by the clocks.
// The closures that read their neighbours' moments (NB) shrink by two sites
// a step: each step's gathered moments go to a second LDS buffer, and the
// update takes the sites whose eight neighbours were gathered.
// The populations pass through the storage codec between the steps, so the
// result equals k single steps bit for bit.  Plain stores: a tile's rows end
// inside cache lines, which the L2 then completes (non-temporal stores
// measured 5-15% slower from 512^2 on).
// KEEP > 0 stores the state after every KEEP steps (k a multiple of it), `stride`
// elements apart from dst on, instead of the last one only.
template <int ST, int EDDY, bool KIN, int RX, int RY, int S, int K, int KEEP = 0, int PH = 1>
__global__ __launch_bounds__(RX* RY / S) void k_tile(
    const typename Codec<ST>::T* __restrict__ src, typename Codec<ST>::T* __restrict__ dst,
    Geom geo, Rates rt, float c12, int steps, int tiles_x, int tile_w, int tile_h,
    long long stride) {
  const int k = K > 0 ? K : steps;
  using C = Codec<ST>;
  using T = typename C::T;
  constexpr bool NB = KIN || EDDY == 2;
  constexpr int NF = KIN ? 5 : 3;     // moments of NB: rho - 1, j (, B)
  constexpr int N = RX * RY, H = RY / S;
  constexpr int NP = 16 / PH;
  __shared__ T pl[NP][N];             // moving planes (kTileRow), PH parts in turn
  __shared__ float mo[NB ? NF : 1][NB ? N : 1];
  const int rx = int(threadIdx.x) % RX, ry0 = int(threadIdx.x) / RX;
  const int halo = NB ? 2 * k - 1 : k - 1;
  // blocks go round-robin to the eight XCDs: each takes a contiguous band of
  // tiles, so that neighbours share halo lines and complete each other's store
  // lines in one L2
  const int tile = (int(blockIdx.x) & 7) * int(gridDim.x >> 3) + (int(blockIdx.x) >> 3);
  const int x0 = (tile % tiles_x) * tile_w, y0 = (tile / tiles_x) * tile_h;
  if (y0 >= geo.ny) return;
  const int wx = min(tile_w, geo.nx - x0), wy = min(tile_h, geo.ny - y0);
  int x = (x0 - halo + rx) % geo.nx;
  x = x < 0 ? x + geo.nx : x;
  const int xl = x == 0 ? geo.nx - 1 : x - 1, xr = x == geo.nx - 1 ? 0 : x + 1;
  float v[S][kNPop][1];
#pragma unroll
  for (int j = 0; j < S; ++j) {
    int y = (y0 - halo + ry0 + j * H) % geo.ny;
    y = y < 0 ? y + geo.ny : y;
    unsigned row[3];
    t2_rows(y, geo, row);
    gather_row<ST, 1>(src, geo.plane, x, xl, xr, row, v[j]);
  }
  auto step = [&](int s) {
    // the update of step s takes the sites at least `in` sites inside the region
    const int in = NB ? 2 * s - 1 : s - 1;
    if constexpr (NB) {
#pragma unroll
      for (int j = 0; j < S; ++j) {
        float p[kNPop], m[5];
#pragma unroll
        for (int q = 0; q < kNPop; ++q) p[q] = v[j][q][0];
        site_moments(p, m);
#pragma unroll
        for (int i = 0; i < NF; ++i) mo[i][(ry0 + j * H) * RX + rx] = m[i];
      }
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const int ry = ry0 + j * H;
      if (rx >= in && rx < RX - in && ry >= in && ry < RY - in) {
        if constexpr (NB) {
          const NbTerms kc = nb_terms<EDDY, KIN>(&mo[0][(ry - 1) * RX], &mo[0][ry * RX],
                                                 &mo[0][(ry + 1) * RX], N, rx, c12);
          float f[9], g[10];
#pragma unroll
          for (int i = 0; i < 9; ++i) f[i] = v[j][i][0];
#pragma unroll
          for (int i = 0; i < 10; ++i) g[i] = v[j][9 + i][0];
          collide<EDDY, KIN>(f, g, rt, kc);
#pragma unroll
          for (int i = 0; i < 9; ++i) v[j][i][0] = f[i];
#pragma unroll
          for (int i = 0; i < 10; ++i) v[j][9 + i][0] = g[i];
        } else {
          collide_sites<1, EDDY == 1, ST == kFP16S>(v[j], rt);
        }
        if constexpr (KEEP > 0) {
          const int oy = ry - halo;
          if (s % KEEP == 0 && s < k && rx >= halo && rx < halo + wx && oy >= 0 && oy < wy)
            store_row<ST, 1, false>(dst + (s / KEEP - 1) * stride, geo.plane,
                                    unsigned(y0 + oy) * geo.pitch + unsigned(x), v[j]);
        }
        if (s < k) {
#pragma unroll
          for (int q = 0; q < kNPop; ++q) {
            if (kTileRow[q] >= NP) continue;   // a later part
            const T e = C::enc(v[j][q][0]);
            if (kTileRow[q] >= 0)
              pl[kTileRow[q] < 0 ? 0 : kTileRow[q]][ry * RX + rx] = e;
            else
              v[j][q][0] = C::dec(e);
          }
        }
      }
    }
    if (s == k) return;
#pragma unroll
    for (int ph = 0; ph < PH; ++ph) {
      if (ph > 0) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < S; ++j) {
          const int ry = ry0 + j * H;
          if (rx >= in && rx < RX - in && ry >= in && ry < RY - in) {
#pragma unroll
            for (int q = 0; q < kNPop; ++q)
              if (kTileRow[q] / NP == ph && kTileRow[q] >= 0)
                pl[kTileRow[q] < 0 ? 0 : kTileRow[q] % NP][ry * RX + rx] = C::enc(v[j][q][0]);
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < S; ++j) {
        const int ry = ry0 + j * H;
        if (rx > in && rx < RX - 1 - in && ry > in && ry < RY - 1 - in) {
#pragma unroll
          for (int q = 0; q < kNPop; ++q)
            if (kTileRow[q] / NP == ph && kTileRow[q] >= 0)
              v[j][q][0] = C::dec(pl[kTileRow[q] < 0 ? 0 : kTileRow[q] % NP]
                                    [(ry - kPlaneCy[q]) * RX + rx - kPlaneCx[q]]);
        }
      }
    }
    if constexpr (!NB) __syncthreads();   // NB: the moments' barrier follows every read
  };
  if constexpr (K > 0) {
#pragma unroll
    for (int s = 1; s <= K; ++s) step(s);
  } else {
    for (int s = 1; s <= k; ++s) step(s);
  }
  if constexpr (KEEP > 0) dst += (k / KEEP - 1) * stride;
  if (rx >= halo && rx < halo + wx) {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const int oy = ry0 + j * H - halo;
      if (oy >= 0 && oy < wy)
        store_row<ST, 1, false>(dst, geo.plane, unsigned(y0 + oy) * geo.pitch + unsigned(x), v[j]);
    }
  }
}

// ------------------------------------------------------ in-place (AA) step
// One lattice updated in place by two alternating steps.  Layout N (natural,
// as for k_step): slot q at x holds the post-collision f*_q(x).  Layout R
// (reversed): slot opp(q) at x + c_q holds f*_q(x).
//   PHASE 0, N -> R: pre_q(x) = N_q(x - c_q), the pull gather of k_step;
//     collide; f*_q(x) is stored in slot opp(q) at x + c_q.
//   PHASE 1, R -> N: pre_q(x) = R_opp(q)(x), all local; collide; f*_q(x) is
//     stored in slot q at x.
// In both phases the locations whose values a thread uses and the locations
// it writes are the same set, and no two threads share one, so no thread
// reads a value another thread writes in the same launch.  (With V = 2 the
// paired loads of x-moving planes also fetch one neighbour element that is
// not used; x-moving planes are stored element by element.)
__device__ constexpr int kPlaneOpp[kNPop] = {0,  3,  4,  1,  2,  7,  8,  5,  6, 9,
                                             12, 13, 10, 11, 14, 17, 18, 15, 16};

template <int ST, int V, bool LES, int PHASE>
__global__ __launch_bounds__(kStepThreads) void k_step_aa(typename Codec<ST>::T* __restrict__ lat,
                                                          Geom geo, Rates rt, int tiles_x) {
  using C = Codec<ST>;
  using T = typename C::T;
  using VT = typename Vec<T, V>::type;
  const int x0 = ((int(blockIdx.x) % tiles_x) * kStepThreads + int(threadIdx.x)) * V;
  const int y = int(blockIdx.x) / tiles_x;
  if (x0 >= geo.nx) return;
  const int xl = x0 == 0 ? geo.nx - 1 : x0 - 1;
  const int xr = x0 + V == geo.nx ? 0 : x0 + V;
  const int ym = y == 0 ? geo.ny - 1 : y - 1;
  const int yp = y == geo.ny - 1 ? 0 : y + 1;
  // row[c + 1] is the row of y - c
  const unsigned row[3] = {unsigned(yp) * geo.pitch, unsigned(y) * geo.pitch,
                           unsigned(ym) * geo.pitch};
  const long long P = geo.plane;
  float v[kNPop][V];
#pragma unroll
  for (int q = 0; q < kNPop; ++q) {
    if (PHASE == 1) {
      const VT a = ld_plane<VT>(lat + kPlaneOpp[q] * P, row[1] + unsigned(x0));
      if constexpr (V == 1) {
        v[q][0] = C::dec(a);
      } else {
#pragma unroll
        for (int j = 0; j < V; ++j) v[q][j] = C::dec(a[j]);
      }
    } else {
      const T* __restrict__ base = lat + q * P;
      const unsigned r = row[kPlaneCy[q] + 1];
      if (V == 1 || kPlaneCx[q] == 0) {
        const int xs = kPlaneCx[q] == 0 ? x0 : (kPlaneCx[q] == 1 ? xl : xr);
        const VT a = ld_plane<VT>(base, r + unsigned(xs));
        if constexpr (V == 1) {
          v[q][0] = C::dec(a);
        } else {
#pragma unroll
          for (int j = 0; j < V; ++j) v[q][j] = C::dec(a[j]);
        }
      } else if constexpr (V > 1) {
        const VT a = ld_plane<VT>(base, r + unsigned(x0));
        const float e = C::dec(ld_plane<T>(base, r + unsigned(kPlaneCx[q] == 1 ? xl : xr)));
#pragma unroll
        for (int j = 0; j < V; ++j) {
          if (kPlaneCx[q] == 1)
            v[q][j] = j == 0 ? e : C::dec(a[j > 0 ? j - 1 : 0]);
          else
            v[q][j] = j == V - 1 ? e : C::dec(a[j < V - 1 ? j + 1 : 0]);
        }
      }
    }
  }
  float out[kNPop][V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    float f[9], g[10];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = v[i][j];
#pragma unroll
    for (int k = 0; k < 10; ++k) g[k] = v[9 + k][j];
    collide<LES ? 1 : 0, false, ST == kFP16S>(f, g, rt);
#pragma unroll
    for (int i = 0; i < 9; ++i) out[i][j] = f[i];
#pragma unroll
    for (int k = 0; k < 10; ++k) out[9 + k][j] = g[k];
  }
#pragma unroll
  for (int q = 0; q < kNPop; ++q) {
    if (PHASE == 1 || kPlaneCx[q] == 0) {
      // local store (PHASE 1), or the unshifted x of a plane moving along y only
      T* __restrict__ base = lat + (PHASE == 1 ? q : kPlaneOpp[q]) * P;
      const unsigned r = PHASE == 1 ? row[1] : row[1 - kPlaneCy[q]];
      VT w;
      if constexpr (V == 1) {
        w = C::enc(out[q][0]);
      } else {
#pragma unroll
        for (int j = 0; j < V; ++j) w[j] = C::enc(out[q][j]);
      }
      st_plane_nt<VT>(base, r + unsigned(x0), w);
    } else {
      // f*_q(x0 + j) goes to x0 + j + c_x: one element at a time
      T* __restrict__ base = lat + kPlaneOpp[q] * P;
      const unsigned r = row[1 - kPlaneCy[q]];
#pragma unroll
      for (int j = 0; j < V; ++j) {
        int xd = x0 + j + kPlaneCx[q];
        xd = xd < 0 ? geo.nx - 1 : (xd >= geo.nx ? xd - geo.nx : xd);
        st_plane_nt<T>(base, r + unsigned(xd), C::enc(out[q][j]));
      }
    }
  }
}

// Layout R -> N in place: for each plane q of one direction of every
// opposite pair (the other is opp(q)), swap slot q at x with slot opp(q) at
// x + c_q.  Each pair of locations belongs to exactly one (x, q), so the
// swaps are independent.  One workgroup per row.
template <int ST>
__global__ __launch_bounds__(256) void k_unswap_aa(typename Codec<ST>::T* __restrict__ lat,
                                                   Geom geo) {
  using T = typename Codec<ST>::T;
  constexpr int kHalf[8] = {1, 2, 5, 6, 10, 11, 15, 16};
  const int y = int(blockIdx.x);
  const long long P = geo.plane;
  for (int x = int(threadIdx.x); x < geo.nx; x += int(blockDim.x)) {
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      const int q = kHalf[h];
      int xd = x + kPlaneCx[q], yd = y + kPlaneCy[q];
      xd = xd < 0 ? geo.nx - 1 : (xd >= geo.nx ? 0 : xd);
      yd = yd < 0 ? geo.ny - 1 : (yd >= geo.ny ? 0 : yd);
      T* a = lat + q * P + (long long)y * geo.pitch + x;
      T* b = lat + kPlaneOpp[q] * P + (long long)yd * geo.pitch + xd;
      const T t = *a;
      *a = *b;
      *b = t;
    }
  }
}

// ------------------------------------------------------- initialisation etc.
// f^eq - w and g^eq of Sec. 3 in FP64 at one site.
__device__ __forceinline__ void equilibrium_dev(double rho, double ux, double uy, double bx,
                                                double by, double (&df)[9], double (&gq)[10]) {
  const double u2 = ux * ux + uy * uy, b2 = bx * bx + by * by;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const double cu = kCx[i] * ux + kCy[i] * uy;
    const double cb = kCx[i] * bx + kCy[i] * by;
    const double c2 = double(kCx[i] * kCx[i] + kCy[i] * kCy[i]);
    df[i] = kW[i] * (rho - 1.0) + kW[i] * rho * (3.0 * cu + 4.5 * cu * cu - 1.5 * u2) +
            4.5 * kW[i] * (0.5 * b2 * c2 - cb * cb);
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const double cu = kMx[k] * ux + kMy[k] * uy;
    const double cb = kMx[k] * bx + kMy[k] * by;
    gq[k] = kWm[k] * (bx + 3.0 * (cu * bx - cb * ux));
    gq[5 + k] = kWm[k] * (by + 3.0 * (cu * by - cb * uy));
  }
}

template <int ST>
__global__ void k_init(const double* __restrict__ rho, const double* __restrict__ ux,
                       const double* __restrict__ uy, const double* __restrict__ bx,
                       const double* __restrict__ by, typename Codec<ST>::T* __restrict__ lat,
                       Geom geo) {
  using C = Codec<ST>;
  const long long n = (long long)geo.nx * geo.ny;
  const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int y = int(s / geo.nx), x = int(s % geo.nx);
  double df[9], gq[10];
  equilibrium_dev(rho[s], ux[s], uy[s], bx[s], by[s], df, gq);
  const long long o = (long long)y * geo.pitch + x;
#pragma unroll
  for (int i = 0; i < 9; ++i) lat[i * geo.plane + o] = C::enc(float(df[i]));
#pragma unroll
  for (int q = 0; q < 10; ++q) lat[(9 + q) * geo.plane + o] = C::enc(float(gq[q]));
}

template <int ST>
__global__ void k_decode(const typename Codec<ST>::T* __restrict__ lat, double* __restrict__ out,
                         Geom geo) {
  using C = Codec<ST>;
  const long long n = (long long)geo.nx * geo.ny;
  const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int y = int(s / geo.nx), x = int(s % geo.nx);
  const long long o = (long long)y * geo.pitch + x;
#pragma unroll
  for (int q = 0; q < kNPop; ++q) {
    const double w = q < 9 ? kW[q] : 0.0;
    out[q * n + s] = w + double(C::dec(lat[q * geo.plane + o]));
  }
}

template <int ST>
__global__ void k_encode(const double* __restrict__ in, typename Codec<ST>::T* __restrict__ lat,
                         Geom geo) {
  using C = Codec<ST>;
  const long long n = (long long)geo.nx * geo.ny;
  const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int y = int(s / geo.nx), x = int(s % geo.nx);
  const long long o = (long long)y * geo.pitch + x;
#pragma unroll
  for (int q = 0; q < kNPop; ++q) {
    const double w = q < 9 ? kW[q] : 0.0;
    lat[q * geo.plane + o] = C::enc(float(in[q * n + s] - w));
  }
}

// Macroscopic fields (FP64) of the stored state at one site; returns false if
// any population is not finite.
template <int ST>
__device__ __forceinline__ bool macro_site(const typename Codec<ST>::T* __restrict__ lat,
                                           const Geom& geo, long long o, double& rho,
                                           double& ux, double& uy, double& bx, double& by) {
  using C = Codec<ST>;
  float v[kNPop];
  bool ok = true;
#pragma unroll
  for (int q = 0; q < kNPop; ++q) {
    v[q] = C::dec(lat[q * geo.plane + o]);
    ok = ok && isfinite(v[q]);
  }
  double dr = 0.0, jx = 0.0, jy = 0.0, b0 = 0.0, b1 = 0.0;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    dr += double(v[i]);
    jx += kCx[i] * double(v[i]);
    jy += kCy[i] * double(v[i]);
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    b0 += double(v[9 + k]);
    b1 += double(v[14 + k]);
  }
  rho = 1.0 + dr;
  ux = jx / rho;
  uy = jy / rho;
  bx = b0;
  by = b1;
  return ok;
}

template <int ST>
__global__ void k_macro(const typename Codec<ST>::T* __restrict__ lat, double* __restrict__ rho,
                        double* __restrict__ ux, double* __restrict__ uy,
                        double* __restrict__ bx, double* __restrict__ by, Geom geo) {
  const long long n = (long long)geo.nx * geo.ny;
  const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int y = int(s / geo.nx), x = int(s % geo.nx);
  double r, a, b, c, d;
  macro_site<ST>(lat, geo, (long long)y * geo.pitch + x, r, a, b, c, d);
  rho[s] = r;
  ux[s] = a;
  uy[s] = b;
  bx[s] = c;
  by[s] = d;
}

template <int ST>
__global__ void k_macro_box(const typename Codec<ST>::T* __restrict__ lat, int w,
                            double* __restrict__ rho, double* __restrict__ ux,
                            double* __restrict__ uy, double* __restrict__ bx,
                            double* __restrict__ by, Geom geo) {
  const int cnx = geo.nx / w, cny = geo.ny / w;
  const long long n = (long long)cnx * cny;
  const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int cy = int(s / cnx), cx = int(s % cnx);
  double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int dy = 0; dy < w; ++dy)
    for (int dx = 0; dx < w; ++dx) {
      double v[5];
      macro_site<ST>(lat, geo, (long long)(cy * w + dy) * geo.pitch + (cx * w + dx), v[0], v[1],
                     v[2], v[3], v[4]);
#pragma unroll
      for (int q = 0; q < 5; ++q) a[q] += v[q];
    }
  const double iw = 1.0 / (double(w) * w);
  rho[s] = a[0] * iw;
  ux[s] = a[1] * iw;
  uy[s] = a[2] * iw;
  bx[s] = a[3] * iw;
  by[s] = a[4] * iw;
}

// Per-block partial sums of |u - u_t|^2 + |B - B_t|^2 (grid-stride over sites).
template <int ST>
__global__ __launch_bounds__(256) void k_mismatch(const typename Codec<ST>::T* __restrict__ lat,
                                                  const double* __restrict__ ux_t,
                                                  const double* __restrict__ uy_t,
                                                  const double* __restrict__ bx_t,
                                                  const double* __restrict__ by_t,
                                                  double* __restrict__ part, Geom geo) {
  __shared__ double sh[256];
  const long long n = (long long)geo.nx * geo.ny;
  double acc = 0.0;
  for (long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x; s < n;
       s += (long long)gridDim.x * blockDim.x) {
    const int y = int(s / geo.nx), x = int(s % geo.nx);
    double r, u, v, b0, b1;
    macro_site<ST>(lat, geo, (long long)y * geo.pitch + x, r, u, v, b0, b1);
    const double du = u - ux_t[s], dv = v - uy_t[s], d0 = b0 - bx_t[s], d1 = b1 - by_t[s];
    acc += du * du + dv * dv + d0 * d0 + d1 * d1;
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_copy(const uint4* __restrict__ src, uint4* __restrict__ dst, long long n16) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
       i += (long long)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// ------------------------------------------------------------ diagnostics
enum {
  kSumMass = 0, kSumMx, kSumMy, kSumBx, kSumBy, kSumEk, kSumEm, kSumHc, kSumOm, kSumJ2,
  kSumBad, kNSum,          // slots 0..10 are sums
  kMaxDiv = kNSum, kMaxU,  // slots 11, 12 are maxima
  kNRed
};

// The sums and maxima of a block of 256 threads into out[0 .. kNRed) (ROOT:
// the square root of the largest |u|^2), reduced through `red` (kNRed x 256
// doubles of LDS): each wave takes every fourth quantity, four values a lane
// from LDS and six exchanges in registers, one barrier in all (a tree of
// eight barriers over all quantities: k_step_diag 10.2 us at 64^2 against 9.5,
// k_diag_final 3.7 against 3.3).  In a block of more WAVES the 256 threads with
// on hand in their values as thread t.
template <bool ROOT, int WAVES = 4>
__device__ __forceinline__ void block_reduce(const double (&v)[kNRed], double* __restrict__ red,
                                             double* __restrict__ out, int t, bool on = true) {
#pragma clang fp contract(off)
  const int lane = int(threadIdx.x) & 63;
  if (on) {
#pragma unroll
    for (int q = 0; q < kNRed; ++q) red[q * 256 + t] = v[q];
  }
  __syncthreads();
  for (int q = int(threadIdx.x) >> 6; q < kNRed; q += WAVES) {
    const double* r = red + q * 256 + lane;
    const double r0 = r[0], r1 = r[64], r2 = r[128], r3 = r[192];
    double a = q < kNSum ? (r0 + r1) + (r2 + r3) : fmax(fmax(r0, r1), fmax(r2, r3));
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
      const double o = __shfl_xor(a, w);
      a = q < kNSum ? a + o : fmax(a, o);
    }
    if (lane == 0) out[q] = ROOT && q == kMaxU ? sqrt(a) : a;
  }
}

// One pass over the lattice: a block of kDiagThreads threads owns as many
// columns and walks strips of `rows` rows (tile t, strip r: unit
// r * tiles_x + t; a block takes units blockIdx.x, + gridDim.x, ...).  Per row
// it loads the populations of row y + 1 (no streaming: the moments of the
// current state), forms rho, u, B in FP64 into a rolling 3-row LDS buffer with
// one halo column on each side, and then accumulates row y: the sums and
// maxima of the site's own fields and the centred differences
// d_x a = (a(x + 1) - a(x - 1)) / 2 of div B, w = d_x u_y - d_y u_x and
// j = d_x B_y - d_y B_x.  A site with a non-finite population has rho = NaN.
// Each block writes one partial (sums, maxima) to part[blockIdx.x], with the
// largest |u|^2 in the slot of max |u|: the final fold takes its square root
// (a correctly rounded square root is monotone, so the root of the largest
// square is the largest root).
constexpr int kDiagThreads = 256;
constexpr int kDiagRows = 64;   // the most rows of a strip

constexpr int kDiagNC = kDiagThreads + 2;
typedef double DiagRing[3][5][kDiagNC];   // rho, ux, uy, Bx, By of three rows

// The moments of one site from its stored populations (deviations f - w in
// the storage order, decoded by C) into column col of ring slot `slot`: rho
// (NaN when a population is not finite), u = j / rho and B.  Contraction is
// off here and in the two functions below, so that every kernel inlining
// them forms the diagnostics identically.
template <class C>
__device__ __forceinline__ void diag_moments(const typename C::T (&p)[kNPop], DiagRing& mac,
                                             int slot, int col) {
#pragma clang fp contract(off)
  bool ok = true;
  double dr = 0.0, jx = 0.0, jy = 0.0, b0 = 0.0, b1 = 0.0;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const float f = C::dec(p[i]);
    ok = ok && isfinite(f);
    dr += double(f);
    jx += kCx[i] * double(f);
    jy += kCy[i] * double(f);
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const float gx = C::dec(p[9 + k]), gy = C::dec(p[14 + k]);
    ok = ok && isfinite(gx) && isfinite(gy);
    b0 += double(gx);
    b1 += double(gy);
  }
  const double r = 1.0 + dr;
  const double ir = 1.0 / r;
  mac[slot][0][col] = ok ? r : __builtin_nan("");
  mac[slot][1][col] = jx * ir;
  mac[slot][2][col] = jy * ir;
  mac[slot][3][col] = b0;
  mac[slot][4][col] = b1;
}

// Adds the site in ring column c of the middle row (slot s0; sm below, sp
// above) to the thread's sums and maxima.
__device__ __forceinline__ void diag_accumulate(double (&v)[kNRed], const DiagRing& mac, int sm,
                                                int s0, int sp, int c) {
#pragma clang fp contract(off)
  const double r = mac[s0][0][c], ux = mac[s0][1][c], uy = mac[s0][2][c];
  const double b0 = mac[s0][3][c], b1 = mac[s0][4][c];
  const double jx = r * ux, jy = r * uy;
  v[kSumMass] += r;
  v[kSumMx] += jx;
  v[kSumMy] += jy;
  v[kSumBx] += b0;
  v[kSumBy] += b1;
  v[kSumEk] += 0.5 * (jx * ux + jy * uy);   // |j|^2 / (2 rho)
  v[kSumEm] += 0.5 * (b0 * b0 + b1 * b1);
  v[kSumHc] += ux * b0 + uy * b1;
  const double div = 0.5 * (mac[s0][3][c + 1] - mac[s0][3][c - 1]) +
                     0.5 * (mac[sp][4][c] - mac[sm][4][c]);
  const double om = 0.5 * (mac[s0][2][c + 1] - mac[s0][2][c - 1]) -
                    0.5 * (mac[sp][1][c] - mac[sm][1][c]);
  const double jz = 0.5 * (mac[s0][4][c + 1] - mac[s0][4][c - 1]) -
                    0.5 * (mac[sp][3][c] - mac[sm][3][c]);
  v[kSumOm] += 0.5 * om * om;
  v[kSumJ2] += 0.5 * jz * jz;
  v[kSumBad] += isfinite(r) ? 0.0 : 1.0;
  v[kMaxDiv] = fmax(v[kMaxDiv], fabs(div));
  v[kMaxU] = fmax(v[kMaxU], ux * ux + uy * uy);   // |u|^2: rooted in the fold
}

// The block's sums and maxima into part[blockIdx.x], reduced in the (idle)
// ring.
__device__ __forceinline__ void diag_partial(const double (&v)[kNRed], DiagRing& mac,
                                             double* __restrict__ part) {
  static_assert(kDiagThreads == 256 && 3 * 5 * kDiagNC >= kNRed * kDiagThreads,
                "ring too small to reduce in");
  block_reduce<false>(v, &mac[0][0][0], part + (long long)blockIdx.x * kDiagSlots,
                      int(threadIdx.x));
}

template <int ST>
__global__ __launch_bounds__(kDiagThreads) void k_diag(const typename Codec<ST>::T* __restrict__ lat,
                                                       double* __restrict__ part, Geom geo,
                                                       int tiles_x, int units, int rows) {
  using C = Codec<ST>;
  using T = typename C::T;
  __shared__ DiagRing mac;
  const int tx = int(threadIdx.x);
  double v[kNRed];
#pragma unroll
  for (int q = 0; q < kNRed; ++q) v[q] = 0.0;
  for (int u = int(blockIdx.x); u < units; u += int(gridDim.x)) {
    const int xt = (u % tiles_x) * kDiagThreads;
    const int y0 = (u / tiles_x) * rows;
    const int y1 = min(y0 + rows, geo.ny);
    const int x = xt + tx;
    const bool active = x < geo.nx;
    const int xc = x % geo.nx;   // past the last column: its periodic images
    const int xh = tx == 0 ? (xt == 0 ? geo.nx - 1 : xt - 1) : (xt + kDiagThreads) % geo.nx;
    const int ch = tx == 0 ? 0 : kDiagNC - 1;
    T raw[kNPop], rawh[kNPop];
    auto load = [&](int xx, int yy, T (&p)[kNPop]) {
      const unsigned o = unsigned(yy) * geo.pitch + unsigned(xx);
#pragma unroll
      for (int q = 0; q < kNPop; ++q) p[q] = ld_plane<T>(lat + q * geo.plane, o);
    };
    auto issue = [&](int yy) {
      yy = yy < 0 ? yy + geo.ny : (yy >= geo.ny ? yy - geo.ny : yy);
      load(xc, yy, raw);
      if (tx < 2) load(xh, yy, rawh);
    };
    auto commit = [&](int slot) {
      diag_moments<C>(raw, mac, slot, tx + 1);
      if (tx < 2) diag_moments<C>(rawh, mac, slot, ch);
    };
    issue(y0 - 1);
    commit(0);
    issue(y0);
    commit(1);
    issue(y0 + 1);
    for (int y = y0; y < y1; ++y) {
      const int sm = (y - y0) % 3, s0 = (y - y0 + 1) % 3, sp = (y - y0 + 2) % 3;
      commit(sp);
      if (y + 2 <= y1) issue(y + 2);
      __syncthreads();
      if (active) diag_accumulate(v, mac, sm, s0, sp, tx + 1);
      __syncthreads();
    }
  }
  diag_partial(v, mac, part);
}

// One step src -> dst (as k_step, FP32 storage) fused with the diagnostics
// of dst (as k_diag): the same tiles, strips, units and accumulation order, so
// the partials equal those of k_diag on the stored result bit for bit.  Each
// block computes the new state of its strip's rows and of the row above and
// below (not stored), on its tile's columns and one halo column on each side
// (threads 0 and 1, not stored), gathering the next row while it accumulates
// the current one; only the strip's own rows and columns are written.
template <bool LES>
__global__ __launch_bounds__(kDiagThreads) void k_step_diag(const float* __restrict__ src,
                                                            float* __restrict__ dst,
                                                            double* __restrict__ part, Geom geo,
                                                            Rates rt, int tiles_x, int units,
                                                            int rows) {
  __shared__ DiagRing mac;
  const int tx = int(threadIdx.x);
  const long long P = geo.plane;
  double v[kNRed];
#pragma unroll
  for (int q = 0; q < kNRed; ++q) v[q] = 0.0;
  for (int u = int(blockIdx.x); u < units; u += int(gridDim.x)) {
    const int xt = (u % tiles_x) * kDiagThreads;
    const int y0 = (u / tiles_x) * rows;
    const int y1 = min(y0 + rows, geo.ny);
    const int x = xt + tx;
    const bool active = x < geo.nx;
    const int xc = x % geo.nx;   // past the last column: its periodic images
    const int xh = tx == 0 ? (xt == 0 ? geo.nx - 1 : xt - 1) : (xt + kDiagThreads) % geo.nx;
    const int ch = tx == 0 ? 0 : kDiagNC - 1;
    const int xcl = xc == 0 ? geo.nx - 1 : xc - 1, xcr = xc == geo.nx - 1 ? 0 : xc + 1;
    const int xhl = xh == 0 ? geo.nx - 1 : xh - 1, xhr = xh == geo.nx - 1 ? 0 : xh + 1;
    float f[kNPop][1], fh[kNPop][1];   // the gathered row in flight
    auto gather = [&](int r) {
      unsigned row[3];
      t2_rows(r, geo, row);
      gather_row<LBMHD_FP32, 1>(src, P, xc, xcl, xcr, row, f);
      if (tx < 2) gather_row<LBMHD_FP32, 1>(src, P, xh, xhl, xhr, row, fh);
    };
    auto moments = [&](const float (&w)[kNPop][1], int slot, int col) {
      float e[kNPop];   // FP32 storage: the values stored are the collided ones
#pragma unroll
      for (int q = 0; q < kNPop; ++q) e[q] = w[q][0];
      diag_moments<Codec<LBMHD_FP32>>(e, mac, slot, col);
    };
    // collide the gathered row r, store it if it is one of the strip's rows,
    // and put its moments into ring slot `slot`
    auto finish = [&](int r, int slot) {
      collide_sites<1, LES, false>(f, rt);
      if (active && r >= y0 && r < y1)
        store_row<LBMHD_FP32, 1>(dst, P, unsigned(r) * geo.pitch + unsigned(x), f);
      moments(f, slot, tx + 1);
      if (tx < 2) {
        collide_sites<1, LES, false>(fh, rt);
        moments(fh, slot, ch);
      }
    };
    gather(y0 - 1);
    finish(y0 - 1, 0);
    gather(y0);
    finish(y0, 1);
    gather(y0 + 1);
    for (int y = y0; y < y1; ++y) {
      const int sm = (y - y0) % 3, s0 = (y - y0 + 1) % 3, sp = (y - y0 + 2) % 3;
      finish(y + 1, sp);
      if (y + 2 <= y1) gather(y + 2);
      __syncthreads();
      if (active) diag_accumulate(v, mac, sm, s0, sp, tx + 1);
      __syncthreads();
    }
  }
  diag_partial(v, mac, part);
}

// Both where each row has a block (diag_by_row): the three rows of the ring at
// once, 256 threads each and six lanes of a last wave for the halo columns,
// so that the chain is one gather, one collision and the moments' FP64 work
// instead of three of each.  The row's sums are taken as above, so the partials
// are the same bit for bit.  Columns past the lattice's right edge but the first
// have nothing to do.
constexpr int kDiagRowThreads = 3 * kDiagThreads + 64;
template <int ST, bool STEP, bool LES>
__global__ __launch_bounds__(kDiagRowThreads) void k_diag_row(
    const typename Codec<ST>::T* __restrict__ src, typename Codec<ST>::T* __restrict__ dst,
    double* __restrict__ part, Geom geo, Rates rt, int tiles_x) {
  using C = Codec<ST>;
  using T = typename C::T;
  __shared__ DiagRing mac;
  const int tid = int(threadIdx.x), k = tid - 3 * kDiagThreads;
  const int xt = (int(blockIdx.x) % tiles_x) * kDiagThreads, y0 = int(blockIdx.x) / tiles_x;
  const int slot = k < 0 ? tid / kDiagThreads : k >> 1;   // row y0 - 1 + slot
  const int tx = tid % kDiagThreads;
  int x = xt + tx;
  bool has = x <= geo.nx;
  int col = tx + 1;
  if (k >= 0) {
    has = k < 6;
    x = (k & 1) == 0 ? (xt == 0 ? geo.nx - 1 : xt - 1) : xt + kDiagThreads;
    col = (k & 1) == 0 ? 0 : kDiagNC - 1;
  }
  const bool own = k < 0 && slot == 1 && x < geo.nx;
  if (has) {
    x %= geo.nx;
    unsigned row[3];
    t2_rows(y0 - 1 + slot, geo, row);
    T p[kNPop];
    if constexpr (STEP) {
      constexpr int SF = ST == LBMHD_FP32 ? LBMHD_FP32 : kFP16S;
      float f[kNPop][1];
      gather_row<SF, 1>(src, geo.plane, x, x == 0 ? geo.nx - 1 : x - 1,
                        x == geo.nx - 1 ? 0 : x + 1, row, f);
      collide_sites<1, LES, SF == kFP16S>(f, rt);
      if (own) store_row<SF, 1, false>(dst, geo.plane, row[1] + unsigned(x), f);
#pragma unroll
      for (int q = 0; q < kNPop; ++q) p[q] = Codec<SF>::enc(f[q][0]);
    } else {
#pragma unroll
      for (int q = 0; q < kNPop; ++q) p[q] = ld_plane<T>(src + q * geo.plane, row[1] + unsigned(x));
    }
    diag_moments<C>(p, mac, slot, col);
  }
  __syncthreads();
  double v[kNRed];
#pragma unroll
  for (int q = 0; q < kNRed; ++q) v[q] = 0.0;
  if (own) diag_accumulate(v, mac, 0, 1, 2, tx + 1);
  __syncthreads();
  block_reduce<false, kDiagRowThreads / 64>(v, &mac[0][0][0],
                                            part + (long long)blockIdx.x * kDiagSlots, tx,
                                            k < 0 && slot == 1);
}

// Pass 3: one block folds the partials.
__global__ __launch_bounds__(256) void k_diag_final(const double* __restrict__ part, int nparts,
                                                    double* __restrict__ out) {
  double v[kNRed];
#pragma unroll
  for (int q = 0; q < kNRed; ++q) v[q] = 0.0;
  for (int b = threadIdx.x; b < nparts; b += blockDim.x) {
#pragma unroll
    for (int q = 0; q < kNSum; ++q) v[q] += part[(long long)b * kDiagSlots + q];
#pragma unroll
    for (int q = kNSum; q < kNRed; ++q) v[q] = fmax(v[q], part[(long long)b * kDiagSlots + q]);
  }
  __shared__ double red[kNRed * 256];
  block_reduce<true>(v, red, out, int(threadIdx.x));
}

// One block; the rounding errors of the additions are summed beside them
// (Knuth's two-sum), so that this sum adds no rounding of its own beyond the last
// bit.  (The terms, a block's FP64 sums over all its steps, carry theirs.)
constexpr int kSumThreads = 1024;
__global__ __launch_bounds__(kSumThreads) void k_sum(const double* __restrict__ in, long long n,
                                                     double* __restrict__ out) {
#pragma clang fp contract(off) reassociate(off)
  __shared__ double sh[kSumThreads], se[kSumThreads];
  double a = 0.0, e = 0.0;
  auto add = [&](double x) {
    const double t = a + x, z = t - a;
    e += (a - (t - z)) + (x - z);
    a = t;
  };
  for (long long i = threadIdx.x; i < n; i += kSumThreads) add(in[i]);
  for (int w = kSumThreads / 2; w > 0; w >>= 1) {
    sh[threadIdx.x] = a;
    se[threadIdx.x] = e;
    __syncthreads();
    if ((int)threadIdx.x < w) {
      add(sh[threadIdx.x + w]);
      e += se[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = isfinite(e) ? a + e : a;
}

inline unsigned blocks_for(long long n, int bs) { return unsigned((n + bs - 1) / bs); }

}  // namespace

// ----------------------------------------------------------------- launchers
// f(std::bool_constant<b>...) of run-time booleans.
template <class F, class... Done>
void with_bools(F&& f, std::tuple<Done...>) {
  std::apply(f, std::tuple<Done...>{});
}
template <class F, class... Done, class... More>
void with_bools(F&& f, std::tuple<Done...>, bool b, More... more) {
  if (b)
    with_bools(f, std::tuple<Done..., std::true_type>{}, more...);
  else
    with_bools(f, std::tuple<Done..., std::false_type>{}, more...);
}
template <class F, class... More>
void with_bools(F&& f, bool b, More... more) {
  with_bools(f, std::tuple<>{}, b, more...);
}

// Non-temporal stores, except where this lattice and the one it was read from
// stay in the 256 MB last-level cache until the next pass: there plain stores
// end as whole lines in it.  us per step, non-temporal / plain: k_step 1024^2
// FP32 31 / 22, 2048 x 1024 FP16 34 / 22, k_step_t3 1280 x 1024 17.7 / 14.3, k_step2
// 1024^2 18.2 / 14.1, k_step_nb2 23.7 / 21.8; beyond it (1448^2 FP32, 318 MB)
// k_step_t3 26.8 / 27.8 and k_step_nb2 44.6 / 46.4, and in the L2s (512^2 FP16,
// 20 MB) k_step 6.2 / 6.8.  Counted in the 128-byte lines that the rows take, which
// is what the cache holds of narrow lattices (16 x 100000 FP16, 61 MB of sites in
// 486 MB of lines: 98 / 131; 72 x 40000 65 / 76).
// A state that is kept (dst one of many, lbmhd_step_store) leaves the cache to
// those after it, so from 80 MB on it goes past: us per state, non-temporal / plain,
// FP32 1024^2 (three states a pass) 21.4 / 26.6, 1000^2 (one) 29.4 / 34.8, 800^2 (97
// MB) 20.7 / 20.2, 724^2 16.3 / 15.7, 640^2 (62 MB) 13.7 / 11.6; FP16 1500^2 35.3 /
// 38.7, 1100^2 (92 MB) 21.0 / 22.4, 1024^2 (80 MB) 16.8 / 14.4.
bool stores_bypass(const Geom& g, size_t esize, bool kept) {
  const double row = double((size_t(g.nx) * esize + 127) / 128 * 128);
  const double bytes = 2.0 * kNPop * row * g.ny;
  return bytes < 30e6 || bytes > (kept ? 80e6 : 240e6);
}

template <int ST, int V>
void launch_step_v(bool les, const void* src, void* dst, const Geom& g, const Rates& r,
                   hipStream_t s, bool kept) {
  using T = typename Codec<ST>::T;
  const int tiles_x = (g.nx / V + kStepThreads - 1) / kStepThreads;
  const dim3 grid(unsigned(tiles_x) * unsigned(g.ny)), block(kStepThreads);
  auto* a = static_cast<const T*>(src);
  auto* b = static_cast<T*>(dst);
  with_bools([&](auto l, auto nt) {
    hipLaunchKernelGGL((k_step<ST, V, l(), nt()>), grid, block, 0, s, a, b, g, r, tiles_x);
  }, les, stores_bypass(g, sizeof(T), kept));
}

// Strips of the two-step kernel, measured on MI355X: FP32 runs best with about
// 512 blocks (2048^2: 32 rows, 4096^2: 128), FP16 with about 4096 (8192^2: 32
// rows, 4096^2 and 2048^2: 8); halo overhead 2 / rows.
static Strips step2_strips(const Geom& g, int storage, int V) {
  const bool fp16 = storage != LBMHD_FP32;   // LBMHD_FP16 or its scaled tag
  const long long tiles_x = (g.nx + kT2Threads * V - 1) / (kT2Threads * V);
  const int hi = fp16 ? 32 : 128;
  return split_rows(tiles_x, g.ny, fp16 ? 4096 : 512, 8, hi, hi);
}

template <int ST, int V>
void launch_step2_v(bool les, const void* src, void* dst, void* mid, const Geom& g,
                    const Rates& r, hipStream_t s) {
  using T = typename Codec<ST>::T;
  const auto [rows, strips, xcd_map] = step2_strips(g, ST, V);
  const int tiles_x = (g.nx + kT2Threads * V - 1) / (kT2Threads * V);
  const dim3 grid(unsigned(tiles_x) * unsigned(strips)), block(kT2Threads);
  auto* a = static_cast<const T*>(src);
  auto* b = static_cast<T*>(dst);
  auto* m = static_cast<T*>(mid);
  const Halos none{nullptr, nullptr, 0};
  const int h = rows;
  const bool xcd = xcd_map;
  with_bools([&](auto l, auto md, auto nt) {
    hipLaunchKernelGGL((k_step2<ST, V, l(), md(), false, nt()>), grid, block, 0, s, a, b, m, g, r,
                       tiles_x, h, xcd, none);
  }, les, m != nullptr, stores_bypass(g, sizeof(T), m != nullptr));
}

template <int ST, int EDDY, bool KIN>
void launch_step_nb_t(const void* src, void* dst, const Geom& g, const Rates& r, float c12,
                      hipStream_t s) {
  using T = typename Codec<ST>::T;
  const int tiles_x = (g.nx + kKinThreads - 1) / kKinThreads;
  const int strips = (g.ny + kKinRows - 1) / kKinRows;
  const dim3 grid(unsigned(tiles_x) * unsigned(strips)), block(kKinThreads);
  hipLaunchKernelGGL((k_step_nb<ST, EDDY, KIN>), grid, block, 0, s, static_cast<const T*>(src),
                     static_cast<T*>(dst), g, r, c12, tiles_x);
}

template <int ST>
hipError_t launch_step_nb_s(int eddy, bool kin, const void* src, void* dst, const Geom& g,
                            const Rates& r, float c12, hipStream_t s) {
  if (kin && eddy == 0)
    launch_step_nb_t<ST, 0, true>(src, dst, g, r, c12, s);
  else if (kin && eddy == 1)
    launch_step_nb_t<ST, 1, true>(src, dst, g, r, c12, s);
  else if (kin && eddy == 2)
    launch_step_nb_t<ST, 2, true>(src, dst, g, r, c12, s);
  else if (!kin && eddy == 2)
    launch_step_nb_t<ST, 2, false>(src, dst, g, r, c12, s);
  else
    return hipErrorInvalidValue;   // no neighbour terms: the plain step applies
  return hipGetLastError();
}

// Strip height of the two-step kernel with lattice gradients (halo overhead
// 6 / rows): as for the three-step kernel, about 512 blocks up to 128-row
// strips, 32-row strips beyond.
static Strips step_nb2_strips(const Geom& g) {
  return split_rows((g.nx + kNb2Cols - 1) / kNb2Cols, g.ny, 512, 8, 128, 32);
}

template <int ST, int EDDY, bool KIN>
void launch_step_nb2_t(const void* src, void* dst, void* mid, const Geom& g, const Rates& r,
                       float c12, hipStream_t s) {
  using T = typename Codec<ST>::T;
  const auto [rows, strips, xcd_map] = step_nb2_strips(g);
  const int tiles_x = (g.nx + kNb2Cols - 1) / kNb2Cols;
  const dim3 grid(unsigned(tiles_x) * unsigned(strips)), block(kNb2Threads);
  auto* a = static_cast<const T*>(src);
  auto* b = static_cast<T*>(dst);
  auto* m = static_cast<T*>(mid);
  const int h = rows;
  const bool xcd = xcd_map;
  with_bools([&](auto md, auto nt) {
    hipLaunchKernelGGL((k_step_nb2<ST, EDDY, KIN, md(), nt()>), grid, block, 0, s, a, b, m, g, r,
                       c12, tiles_x, h, xcd);
  }, m != nullptr, stores_bypass(g, sizeof(T), m != nullptr));
}

template <int ST>
hipError_t launch_step_nb2_s(int eddy, bool kin, const void* src, void* dst, void* mid,
                             const Geom& g, const Rates& r, float c12, hipStream_t s) {
  if (kin && eddy == 0)
    launch_step_nb2_t<ST, 0, true>(src, dst, mid, g, r, c12, s);
  else if (kin && eddy == 1)
    launch_step_nb2_t<ST, 1, true>(src, dst, mid, g, r, c12, s);
  else if (kin && eddy == 2)
    launch_step_nb2_t<ST, 2, true>(src, dst, mid, g, r, c12, s);
  else if (!kin && eddy == 2)
    launch_step_nb2_t<ST, 2, false>(src, dst, mid, g, r, c12, s);
  else
    return hipErrorInvalidValue;   // no neighbour terms: the plain kernels apply
  return hipGetLastError();
}

hipError_t launch_step_nb2(int storage, int eddy, bool kin, const void* src, void* dst,
                           void* mid, const Geom& g, const Rates& r, double delta,
                           hipStream_t s) {
  const float c12 = float(delta * delta / 12.0);
  if (storage == LBMHD_FP32)
    return launch_step_nb2_s<LBMHD_FP32>(eddy, kin, src, dst, mid, g, r, c12, s);
  return launch_step_nb2_s<LBMHD_FP16>(eddy, kin, src, dst, mid, g, r, c12, s);
}

bool step_nb2_pays(const Geom& g) {
  const long long tiles_x = (g.nx + kNb2Cols - 1) / kNb2Cols;
  return tiles_x * ((g.ny + 7) / 8) >= 512;
}

hipError_t launch_step_nb(int storage, int eddy, bool kin, const void* src, void* dst,
                          const Geom& g, const Rates& r, double delta, hipStream_t s) {
  const float c12 = float(delta * delta / 12.0);
  if (storage == LBMHD_FP32) return launch_step_nb_s<LBMHD_FP32>(eddy, kin, src, dst, g, r, c12, s);
  return launch_step_nb_s<LBMHD_FP16>(eddy, kin, src, dst, g, r, c12, s);
}

hipError_t launch_step(int storage, bool les, const void* src, void* dst, const Geom& g,
                       const Rates& r, hipStream_t s, bool kept) {
  if (storage == LBMHD_FP32)
    launch_step_v<LBMHD_FP32, 1>(les, src, dst, g, r, s, kept);
  else if (g.nx % 2 == 0)
    launch_step_v<kFP16S, 2>(les, src, dst, g, r, s, kept);
  else
    launch_step_v<kFP16S, 1>(les, src, dst, g, r, s, kept);
  return hipGetLastError();
}

bool step2_pays(int storage, const Geom& g) {
  const int V = storage == LBMHD_FP16 && g.nx % 2 == 0 ? 2 : 1;
  const long long tiles_x = (g.nx + kT2Threads * V - 1) / (kT2Threads * V);
  return tiles_x * ((g.ny + 7) / 8) >= 512;
}

// Strip height of the three-step kernel (halo overhead 4 / rows), measured:
// about 512 blocks, which all run at once (registers admit four per CU), up
// to 128-row strips (2048^2: 32 rows, 4096^2: 128; 64-row strips there, 1024
// blocks, were slower); on larger lattices 32-row strips (8192^2: 16-row
// strips as fast, 64 and 8 rows 3% and 8% slower).
static Strips step_t3_strips(const Geom& g) {
  return split_rows((g.nx + kT3Cols - 1) / kT3Cols, g.ny, 512, 8, 128, 32);
}

hipError_t launch_step_t3(bool les, const void* src, void* dst, void* mid1, void* mid2,
                          const Geom& g, const Rates& r, hipStream_t s) {
  const auto [rows, strips, xcd_map] = step_t3_strips(g);
  const int tiles_x = (g.nx + kT3Cols - 1) / kT3Cols;
  const dim3 grid(unsigned(tiles_x) * unsigned(strips)), block(kT3Threads);
  auto* a = static_cast<const float*>(src);
  auto* b = static_cast<float*>(dst);
  auto* m1 = static_cast<float*>(mid1);
  auto* m2 = static_cast<float*>(mid2);
  const Halos none{nullptr, nullptr, 0};
  const int h = rows;
  const bool xcd = xcd_map;
  with_bools([&](auto l, auto md, auto nt) {
    hipLaunchKernelGGL((k_step_t3<l(), md(), false, nt()>), grid, block, 0, s, a, b, m1, m2, g, r,
                       tiles_x, h, xcd, none);
  }, les, m1 != nullptr, stores_bypass(g, 4, m1 != nullptr));
  return hipGetLastError();
}

hipError_t launch_step2(int storage, bool les, const void* src, void* dst, void* mid,
                        const Geom& g, const Rates& r, hipStream_t s) {
  if (storage == LBMHD_FP32)
    launch_step2_v<LBMHD_FP32, 1>(les, src, dst, mid, g, r, s);
  else if (g.nx % 2 == 0)
    launch_step2_v<kFP16S, 2>(les, src, dst, mid, g, r, s);
  else
    launch_step2_v<kFP16S, 1>(les, src, dst, mid, g, r, s);
  return hipGetLastError();
}

// Regions of the tile kernel.  The smallest lattices need blocks, so 16 x 16
// sites and up to five steps (tiles of 8 x 8; closures with neighbour terms
// three steps, 6 x 6); from 200^2 on 32 x 32 (32 x 28 with FP32 neighbour
// terms), two sites a thread: eight waves, two on each SIMD, and two blocks
// per CU in 64-75 KB of LDS each; on large lattices 64 x 32 (launch_tile_wide).
// Regions whose waves do not divide evenly over the SIMDs (40 x 32, 32 x 36,
// 48 x 24) ran at 75k MLUPS at 4096^2 FP32 against 119k, four sites a thread of
// 32 x 32 at 109k, and blocks that stay for several tiles and gather the next
// one ahead at 85k.
template <int ST, int EDDY, bool KIN>
struct Tile {
  static constexpr bool kNb = KIN || EDDY == 2;
  static constexpr int kBigRows = kNb && ST == LBMHD_FP32 ? 28 : 32;
};

static bool tile_small(const Geom& g) { return (long long)g.nx * g.ny <= 40000; }

// Lanes that issue for each site that counts, in regions of rx x ry sites of
// which a rim of `halo` is halo.
static double tile_lanes(const Geom& g, int rx, int ry, int halo) {
  const int w = rx - 2 * halo, h = ry - 2 * halo;
  return double((g.nx + w - 1) / w) * rx * ((g.ny + h - 1) / h) * ry / (double(g.nx) * g.ny);
}

// Steps per launch: without neighbour terms up to nine in the larger region
// while the smaller tiles still leave a CU each (256^2: five steps 14.5 us, 121
// blocks; nine steps 21.3 us, 256 blocks).
static int tile_most(bool nb, const Geom& g) {
  if (nb) return 3;
  int k = 5;
  if (!tile_small(g) && (long long)g.nx * g.ny < 100000)
    for (; k < 9; ++k) {
      const int w = 32 - 2 * k;   // tile of k + 1 steps
      if ((long long)((g.nx + w - 1) / w) * ((g.ny + w - 1) / w) > 256) break;
    }
  return k;
}

// Steps of the launches that keep every state (NB) or every second one.
template <bool NB, int S>
constexpr int kTileKeep = !NB ? 4 : (S == 1 ? 3 : 2);

template <int ST, int EDDY, bool KIN, int RX, int RY, int S, int K, int KEEP = 0, int PH = 1>
static void launch_tile_k(const void* src, void* dst, int k, size_t keep, const Geom& g,
                          const Rates& r, float c12, hipStream_t s) {
  using T = typename Codec<ST>::T;
  const int halo = Tile<ST, EDDY, KIN>::kNb ? 2 * k - 1 : k - 1;
  const int w = RX - 2 * halo, h = RY - 2 * halo;
  const int tiles_x = (g.nx + w - 1) / w, tiles_y = (g.ny + h - 1) / h;
  hipLaunchKernelGGL((k_tile<ST, EDDY, KIN, RX, RY, S, K, KEEP, PH>),
                     dim3((tiles_x * tiles_y + 7) / 8 * 8), dim3(RX * RY / S), 0, s,
                     static_cast<const T*>(src), static_cast<T*>(dst), g, r, c12, k, tiles_x, w, h,
                     (long long)(keep / sizeof(T)));
}

template <int ST, int EDDY, bool KIN, int RX, int RY, int S>
static void launch_tile_r(const void* src, void* dst, int k, size_t keep, const Geom& g,
                          const Rates& r, float c12, hipStream_t s) {
  constexpr bool kNb = Tile<ST, EDDY, KIN>::kNb;
  // the usual count of each kind is compiled for itself: unrolled, no value is
  // moved between registers from step to step (FP16 10-17% faster)
  constexpr int kFull = !kNb ? 5 : (ST == LBMHD_FP32 || S == 1 ? 3 : 2);
  if (keep)
    launch_tile_k<ST, EDDY, KIN, RX, RY, S, kTileKeep<kNb, S>, kNb ? 1 : 2>(src, dst, k, keep, g,
                                                                            r, c12, s);
  else if (k == kFull)
    launch_tile_k<ST, EDDY, KIN, RX, RY, S, kFull>(src, dst, k, keep, g, r, c12, s);
  else
    launch_tile_k<ST, EDDY, KIN, RX, RY, S, 0>(src, dst, k, keep, g, r, c12, s);
}

// 64 x 32 sites, four a thread, for launches of four and five steps of large
// lattices (no neighbour terms): a wave is a row of 64 columns, of which fewer
// are halo (1.4 lanes issue for each site that counts, 1.6 with 32 x 32).
// FP32 passes the planes in two parts through 64 KB of LDS, so that two blocks
// share a CU here too (all at once, one block: 89k MLUPS at 4096^2 against 119k).
// us per step of five, 32 x 32 / 64 x 32: FP32 1200^2 13.1 / 13.2, 1448^2 20.1 /
// 18.7, 2048^2 39.1 / 36.2, 4096^2 155 / 130, 8192^2 606 / 504; FP16 2048^2 31.6 /
// 31.2, 2500^2 48.1 / 46.6, 4096^2 129 / 116, 8192^2 535 / 461.  Keeping every
// second state FP32 1024^2 17.6 / 16.1, 1200^2 26.3 / 24.2, 724^2 8.7 / 8.7.
// Not faster: six steps (FP32 4096^2 132), four parts or six sites a thread
// (more than 128 registers a lane: 220); lattices whose width leaves the wide tiles
// emptier, five steps 32 x 32 / 64 x 32: FP32 60 x 33333 21.6 / 25.9, 72 x 27777 22.4 /
// 25.1, 120 x 50000 55 / 61, FP16 60 x 100000 54 / 76, 72 x 83333 50 / 68.
bool tile_wide(int storage, int k, bool keep, const Geom& g) {
  const double sites = double(g.nx) * g.ny;
  if (keep ? storage != LBMHD_FP32 || sites < 8e5
           : (k != 4 && k != 5) || sites < (storage == LBMHD_FP32 ? 1.6e6 : 5e6))
    return false;
  return 1.02 * tile_lanes(g, 64, 32, k - 1) <= tile_lanes(g, 32, 32, k - 1);
}

template <int ST, int EDDY>
static void launch_tile_wide(const void* src, void* dst, int k, size_t keep, const Geom& g,
                             const Rates& r, float c12, hipStream_t s) {
  constexpr int PH = ST == LBMHD_FP32 ? 2 : 1;
  if (keep) {
    if constexpr (ST == LBMHD_FP32)
      launch_tile_k<ST, EDDY, false, 64, 32, 4, 4, 2, PH>(src, dst, k, keep, g, r, c12, s);
  } else if (k == 5) {
    launch_tile_k<ST, EDDY, false, 64, 32, 4, 5, 0, PH>(src, dst, k, keep, g, r, c12, s);
  } else {
    launch_tile_k<ST, EDDY, false, 64, 32, 4, 4, 0, PH>(src, dst, k, keep, g, r, c12, s);
  }
}

template <int ST, int EDDY, bool KIN>
static void launch_tile_c(const void* src, void* dst, int k, size_t keep, const Geom& g,
                          const Rates& r, float c12, hipStream_t s) {
  if constexpr (!Tile<ST, EDDY, KIN>::kNb)
    if (tile_wide(ST == LBMHD_FP32 ? LBMHD_FP32 : LBMHD_FP16, k, keep > 0, g))
      return launch_tile_wide<ST, EDDY>(src, dst, k, keep, g, r, c12, s);
  if (tile_small(g))
    launch_tile_r<ST, EDDY, KIN, 16, 16, 1>(src, dst, k, keep, g, r, c12, s);
  else
    launch_tile_r<ST, EDDY, KIN, 32, Tile<ST, EDDY, KIN>::kBigRows, 2>(src, dst, k, keep, g, r,
                                                                       c12, s);
}

template <int ST>
static hipError_t launch_tile_s(int eddy, bool kin, const void* src, void* dst, int k, size_t keep,
                                const Geom& g, const Rates& r, float c12, hipStream_t s) {
  constexpr int SN = ST == kFP16S ? LBMHD_FP16 : ST;   // codec of the closures with neighbours
  if (kin && eddy == 0)
    launch_tile_c<SN, 0, true>(src, dst, k, keep, g, r, c12, s);
  else if (kin && eddy == 1)
    launch_tile_c<SN, 1, true>(src, dst, k, keep, g, r, c12, s);
  else if (kin)
    launch_tile_c<SN, 2, true>(src, dst, k, keep, g, r, c12, s);
  else if (eddy == 2)
    launch_tile_c<SN, 2, false>(src, dst, k, keep, g, r, c12, s);
  else if (eddy == 1)
    launch_tile_c<ST, 1, false>(src, dst, k, keep, g, r, c12, s);
  else
    launch_tile_c<ST, 0, false>(src, dst, k, keep, g, r, c12, s);
  return hipGetLastError();
}

hipError_t launch_tile(int storage, int eddy, bool kin, const void* src, void* dst, int k,
                       const Geom& g, const Rates& r, double delta, hipStream_t s, size_t keep) {
  const bool nb = kin || eddy == 2;
  if (k < 1 || k > tile_most(nb, g) || (keep && k != tile_keep(nb, g)))
    return hipErrorInvalidValue;
  const float c12 = float(delta * delta / 12.0);
  if (storage == LBMHD_FP32)
    return launch_tile_s<LBMHD_FP32>(eddy, kin, src, dst, k, keep, g, r, c12, s);
  return launch_tile_s<kFP16S>(eddy, kin, src, dst, k, keep, g, r, c12, s);
}

int tile_keep(bool nb, const Geom& g) {
  if (tile_small(g)) return nb ? kTileKeep<true, 1> : kTileKeep<false, 1>;
  return nb ? kTileKeep<true, 2> : kTileKeep<false, 2>;
}

// The lattice's sites, weighted by the share of the row-walking kernels'
// 256-column tiles that they fill.
static double tile_size(const Geom& g) {
  const double cols = double((g.nx + 255) / 256) * 256;
  return double(g.nx) * g.ny * (g.nx / cols);
}

// The region of a launch of k steps and its halo.
struct Region {
  int rx, ry, halo;
};
static Region tile_region(int storage, bool nb, int k, bool keep, const Geom& g) {
  const int halo = nb ? 2 * k - 1 : k - 1;
  if (!nb && tile_wide(storage, k, keep, g)) return Region{64, 32, halo};
  if (tile_small(g)) return Region{16, 16, halo};
  return Region{32, nb && storage == LBMHD_FP32 ? 28 : 32, halo};
}

// The share of the tiles of a launch of k steps that the lattice fills, relative
// to what it fills of the row-walking kernels' columns.
static double tile_fill(int storage, bool nb, int k, bool keep, const Geom& g) {
  const Region r = tile_region(storage, nb, k, keep, g);
  const int w = r.rx - 2 * r.halo, h = r.ry - 2 * r.halo;
  const double cols = double((g.nx + 255) / 256) * 256;
  return double(r.rx) * r.ry / (double(w) * h * tile_lanes(g, r.rx, r.ry, r.halo)) *
         (cols / g.nx);
}

// Whether that is enough: low, wide lattices leave most of their tiles' rows
// empty, which matters the more, the more of the launch is bound by its lanes and
// not by its latency.  us per step by rows / in tiles: five steps FP32 25000 x 4
// (share 0.17) 4.9 / 5.6, 16666 x 6 (0.25) 4.9 / 3.9, 50000 x 6 (0.25) 7.6 / 9.8, 30000 x 10
// (0.42) 8.7 / 6.2, 83332 x 12 (0.5) 13.9 / 15.2, 31250 x 32 (0.67) 13.0 / 13.3, 107142 x 28
// (0.58) 36.2 / 36.9, 93750 x 32 (0.67) 39 / 33; FP16 37500 x 8 (0.33) 7.2 / 7.8, 93750 x 32
// (0.67) 28.5 / 31.9, 53570 x 56 (0.78) 30.7 / 27.9; neighbour terms FP32 three steps
// 25000 x 4 (0.22) 11.2 / 8.7, 50000 x 6 (0.33) 14.5 / 16.4, 41666 x 24 (0.67) 23.3 / 28.0,
// 20832 x 48 (0.89) 23.4 / 22.2; FP16 two steps 62500 x 16 (0.62) 24.3 / 23.1, 53570 x 56
// (0.72) 62.2 / 56.6 (cross-helicity 62.6 / 66.4), 107142 x 28 (0.54) 54.9 / 74.1;
// kept pairs FP16 53570 x 56 (0.72) 33.2 / 38.0.
static bool tile_filled(int storage, bool nb, int k, bool keep, const Geom& g) {
  const bool fp32 = storage == LBMHD_FP32;
  const double grow = nb ? 0.22 : (fp32 ? 0.19 : 0.27);
  const double top = nb || keep ? (fp32 ? 0.8 : 0.75) : (fp32 ? 0.65 : 0.7);
  return tile_fill(storage, nb, k, keep, g) >=
         std::min(top, grow * std::sqrt(double(g.nx) * g.ny / 1e5));
}

// Which launches go to tiles where these are filled, us per step in tiles / by
// rows.  Five steps: FP32 1024^2 10.2 / 11.7 (k_step_t3), 2048^2 36 / 45, 4096^2 130 / 167,
// 8192 x 4096 252 / 373; FP16 1024^2 9.2 / 12.9 (k_step), 4096^2 116 / 151
// (k_step2), 8192 x 4096 230 / 289.  Neighbour terms, FP32: three steps 724^2
// 11.4 / 20.2 (k_step_nb2), 1300^2 34 / 40, 1448^2 45.1 / 44.5, 2048^2 89 / 73;
// FP16: two steps 1024^2 17.9 / 35 (k_step_nb; three 19.3), 4096^2 237 / 268
// (three 278), 6000^2 510 / 561, 8192^2 1087 / 1070; cross-helicity alone 3000^2
// 147.5 / 156.4, 3500^2 198.6 / 194.7, 4096^2 271 / 266, 8192^2 1111 / 1050, with the
// kinetic closure 1224 / 1437.
int tile_steps(int storage, int eddy, bool kin, const Geom& g) {
  const bool nb = kin || eddy == 2;
  int k = tile_most(nb, g);
  if (nb && storage == LBMHD_FP32 && tile_size(g) >= 1.6e6) return 0;
  if (nb && storage == LBMHD_FP16) {
    if (!(kin && eddy == 2) && tile_size(g) >= (kin ? 5e7 : 1.05e7)) return 0;
    k = tile_size(g) < 4e5 ? 3 : 2;
  }
  return tile_filled(storage, nb, k, false, g) ? k : 0;
}

// Fewer steps.  FP32: four 4096^2 154 / 234 (a triple and a single step), three
// 1448^2 29.1 / 27.0 (k_step_t3), 4096^2 218 / 167, two 724^2 8.5 / 11.3 (k_step2),
// 1024^2 14.3 / 14.2; FP16: three 4096^2 132 / 175, two 1448^2 16.6 / 25.3,
// 2048^2 44.6 / 45.5, 4096^2 180 / 152; one with neighbour terms 1448^2
// 79 / 95 FP32 and 36 / 60 FP16, 2048^2 170 / 132 and 94 / 78.
bool tile_short_pays(int storage, bool nb, int k, const Geom& g) {
  if (!tile_filled(storage, nb, k, false, g)) return false;
  const double fill = std::min(1.0, tile_fill(storage, nb, k, false, g));
  if (nb) return k > 1 || tile_size(g) < 2.2e6 * fill;
  if (k >= (storage == LBMHD_FP32 ? 4 : 3)) return true;
  return k > 1 && (tile_small(g) || fill >= 0.65) &&
         tile_size(g) < (storage == LBMHD_FP32 ? 1.04e6 : 4.0e6) * fill;
}

// Launches that keep states on the way, us per step against the launches that
// keep one each.  Every second state: FP32 64^2 1.4 / 2.2, 512^2 4.5 / 5.7 (two
// steps in tiles), 1024^2 16.1 / 19.2, 1200^2 24.2 / 29.9 (k_step2), 1448^2 38.5 / 37.0;
// FP16 512^2 4.2 / 5.3, 1024^2 10.1 / 11.3, 2048^2 42.3 / 45.6 (k_step2), 2896^2 84
// / 82 (eight steps a launch 20 / 20 at 1024^2 FP32, 60 / 46 at 2048^2 FP16).
// Every state, neighbour terms: FP32 64^2 2.1 / 4.0 (one step in tiles), 512^2
// 8.2 / 10.9, 724^2 16.9 / 18.6, 1024^2 35.6 / 31.8 (k_step_nb2); FP16 512^2 8.5 /
// 9.9, 1024^2 22.4 / 23.3, 1448^2 46.2 / 47.4, 2048^2 89 / 79 (k_step_nb).
bool tile_keep_pays(int storage, bool nb, const Geom& g) {
  const int k = tile_keep(nb, g);
  if (!tile_filled(storage, nb, k, true, g)) return false;
  const double size = tile_size(g) / std::min(1.0, tile_fill(storage, nb, k, true, g));
  if (nb) return size < (storage == LBMHD_FP32 ? 8e5 : 2.2e6);
  return size < (storage == LBMHD_FP32 ? 1.5e6 : 5e6);
}

// ------------------------------------------ several steps in place
// Strips of 32 to 128 rows and tiles of 256 columns: the copies are
// 6 / rows + 8 / 256 of the lattice (8% at 4096^2).
static Strips halo_strips(const Geom& g) {
  return split_rows((g.nx + kT2Threads - 1) / kT2Threads, g.ny, 512, 32, 128, 128, 1);
}

// Against the AA steps, us per step: 2048 x 1024 46.3 / 46.3 by rows, 2048^2
// 66.6 / 108.6, 4096^2 232 / 494 (k_step_t3 0.59 ms a launch, 0.50 on two
// lattices, where no lane takes other addresses than its neighbours; the
// copies 0.10), 8192 x 4096 576 / 1001.  FP16 pairs measured slower than the AA
// steps (276 / 252 us at 4096^2: 32-row strips of two sites a thread, whose
// halo sites wait for the copies, against 8-row strips on two lattices).  256
// columns keep the copies' offsets within 32 bits on every lattice that
// create accepts.
bool inplace_rows_pay(const Geom& g) {
  return g.nx >= kT2Threads && (long long)g.nx * g.ny >= 3000000;
}

// Elements of the saved rows (three a side, of which the pairs use two).
static size_t halo_row_elems(const Geom& g) {
  const int rows = halo_strips(g).rows;
  return size_t((g.ny + rows - 1) / rows) * kNPop * 6 * g.pitch;
}

// At most a quarter of the lattice: six rows a strip are 3/16 of the strips of 32
// rows but three lattices on two rows, where half the memory, which the mode is
// for, would be lost.
size_t inplace_halo_bytes(const Geom& g) {
  if (!inplace_rows_pay(g)) return 0;
  const size_t cols = size_t((g.nx + kT2Threads - 1) / kT2Threads) * kNPop * g.ny * 8;
  const size_t bytes = (halo_row_elems(g) + cols) * sizeof(float) / 256 * 256 + 256;
  return bytes <= kNPop * size_t(g.plane) * sizeof(float) / 4 ? bytes : 0;
}

template <bool LES>
static void launch_inplace_l(int k, float* lat, float* halo, const Geom& g, const Rates& r,
                             hipStream_t s) {
  const auto [rows, strips, xcd_map] = halo_strips(g);
  const int tiles_x = (g.nx + kT2Threads - 1) / kT2Threads, n = (g.ny + rows - 1) / rows;
  const int col_blocks = (g.ny + 31) / 32;
  float* cols = halo + halo_row_elems(g);
  hipLaunchKernelGGL(k_halo_save, dim3(n * kNPop * 2 * k + tiles_x * col_blocks), dim3(256), 0, s,
                     lat, halo, cols, g, k, rows, n, kT2Threads, col_blocks);
  const Halos hs{halo, cols, n};
  const dim3 grid(unsigned(tiles_x) * unsigned(strips));
  float* none = nullptr;
  if (k == 3)
    hipLaunchKernelGGL((k_step_t3<LES, false, true, true>), grid, dim3(kT3Threads), 0, s, lat, lat, none,
                       none, g, r, tiles_x, rows, xcd_map, hs);
  else
    hipLaunchKernelGGL((k_step2<LBMHD_FP32, 1, LES, false, true, true>), grid, dim3(kT2Threads), 0, s,
                       lat, lat, none, g, r, tiles_x, rows, xcd_map, hs);
}

hipError_t launch_inplace_steps(bool les, int k, void* lat, void* halo, const Geom& g,
                                const Rates& r, hipStream_t s) {
  if (k != 2 && k != 3) return hipErrorInvalidValue;
  if (les)
    launch_inplace_l<true>(k, static_cast<float*>(lat), static_cast<float*>(halo), g, r, s);
  else
    launch_inplace_l<false>(k, static_cast<float*>(lat), static_cast<float*>(halo), g, r, s);
  return hipGetLastError();
}

template <int ST, int V, int PHASE>
void launch_step_aa_v(bool les, void* lat, const Geom& g, const Rates& r, hipStream_t s) {
  using T = typename Codec<ST>::T;
  const int tiles_x = (g.nx / V + kStepThreads - 1) / kStepThreads;
  const dim3 grid(unsigned(tiles_x) * unsigned(g.ny)), block(kStepThreads);
  auto* a = static_cast<T*>(lat);
  if (les)
    hipLaunchKernelGGL((k_step_aa<ST, V, true, PHASE>), grid, block, 0, s, a, g, r, tiles_x);
  else
    hipLaunchKernelGGL((k_step_aa<ST, V, false, PHASE>), grid, block, 0, s, a, g, r, tiles_x);
}

// Both steps keep the widths of k_step: 1 FP32 or 2 FP16 sites per thread
// (16-byte vectors in the local step measured slower: 0.534 against 0.482
// ms per FP32 step at 4096^2, the register cost halving the occupancy).
template <int ST, int V>
void launch_step_aa_p(bool les, int phase, void* lat, const Geom& g, const Rates& r,
                      hipStream_t s) {
  if (phase == 0)
    launch_step_aa_v<ST, V, 0>(les, lat, g, r, s);
  else
    launch_step_aa_v<ST, V, 1>(les, lat, g, r, s);
}

hipError_t launch_step_aa(int storage, bool les, int phase, void* lat, const Geom& g,
                          const Rates& r, hipStream_t s) {
  if (storage == LBMHD_FP32)
    launch_step_aa_p<LBMHD_FP32, 1>(les, phase, lat, g, r, s);
  else if (g.nx % 2 == 0)
    launch_step_aa_p<kFP16S, 2>(les, phase, lat, g, r, s);
  else
    launch_step_aa_p<kFP16S, 1>(les, phase, lat, g, r, s);
  return hipGetLastError();
}

hipError_t launch_unswap_aa(int storage, void* lat, const Geom& g, hipStream_t s) {
  const unsigned nb = unsigned(g.ny);
  if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_unswap_aa<LBMHD_FP32>, dim3(nb), dim3(256), 0, s,
                       static_cast<float*>(lat), g);
  else
    hipLaunchKernelGGL(k_unswap_aa<LBMHD_FP16>, dim3(nb), dim3(256), 0, s,
                       static_cast<_Float16*>(lat), g);
  return hipGetLastError();
}

hipError_t launch_init(int storage, const double* rho, const double* ux, const double* uy,
                       const double* bx, const double* by, void* lat, const Geom& g,
                       hipStream_t s) {
  const unsigned nb = blocks_for((long long)g.nx * g.ny, 256);
  if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_init<LBMHD_FP32>, dim3(nb), dim3(256), 0, s, rho, ux, uy, bx, by,
                       static_cast<float*>(lat), g);
  else
    hipLaunchKernelGGL(k_init<LBMHD_FP16>, dim3(nb), dim3(256), 0, s, rho, ux, uy, bx, by,
                       static_cast<_Float16*>(lat), g);
  return hipGetLastError();
}

hipError_t launch_decode(int storage, const void* lat, double* out, const Geom& g,
                         hipStream_t s) {
  const unsigned nb = blocks_for((long long)g.nx * g.ny, 256);
  if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_decode<LBMHD_FP32>, dim3(nb), dim3(256), 0, s,
                       static_cast<const float*>(lat), out, g);
  else
    hipLaunchKernelGGL(k_decode<LBMHD_FP16>, dim3(nb), dim3(256), 0, s,
                       static_cast<const _Float16*>(lat), out, g);
  return hipGetLastError();
}

hipError_t launch_encode(int storage, const double* in, void* lat, const Geom& g,
                         hipStream_t s) {
  const unsigned nb = blocks_for((long long)g.nx * g.ny, 256);
  if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_encode<LBMHD_FP32>, dim3(nb), dim3(256), 0, s, in,
                       static_cast<float*>(lat), g);
  else
    hipLaunchKernelGGL(k_encode<LBMHD_FP16>, dim3(nb), dim3(256), 0, s, in,
                       static_cast<_Float16*>(lat), g);
  return hipGetLastError();
}

hipError_t launch_macro(int storage, const void* lat, double* rho, double* ux, double* uy,
                        double* bx, double* by, const Geom& g, hipStream_t s) {
  const unsigned nb = blocks_for((long long)g.nx * g.ny, 256);
  if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_macro<LBMHD_FP32>, dim3(nb), dim3(256), 0, s,
                       static_cast<const float*>(lat), rho, ux, uy, bx, by, g);
  else
    hipLaunchKernelGGL(k_macro<LBMHD_FP16>, dim3(nb), dim3(256), 0, s,
                       static_cast<const _Float16*>(lat), rho, ux, uy, bx, by, g);
  return hipGetLastError();
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
  const long long n16 = (long long)(bytes / 16);
  const unsigned nb = unsigned(n16 < 256LL * 4096 ? blocks_for(n16, 256) : 4096u);
  if (n16 > 0)
    hipLaunchKernelGGL(k_copy, dim3(nb), dim3(256), 0, s, static_cast<const uint4*>(src),
                       static_cast<uint4*>(dst), n16);
  return hipGetLastError();
}

// Strips of the diagnostics passes.  A block takes its rows one after another
// (about 1.9 us a row, the latency of the loads and of the FP64 chain), so a
// strip is as short as leaves whole strips for 512 blocks with FP32 storage and
// 1024 with FP16, which has half the bytes in flight a row; never a few blocks
// over that, which would run a round of their own.  us of lbmhd_diag, 64-row
// strips / 1024 strips rounded up / this rule: FP32 512^2 106 / 45 / 40, 1024^2 105 /
// 57 / 49, 2500^2 135 / 149 / 122, 100000 x 8 45 / 55 / 45; FP16 1024^2 119 / 49 /
// 49, 2500^2 142 / 120 / 99, 100000 x 8 47 / 50 / 46.  On the largest lattices 64
// rows are 8-11% faster than 16 (two halo rows a strip).
int diag_rows(int storage, const Geom& g) {
  const int tiles_x = (g.nx + kDiagThreads - 1) / kDiagThreads;
  const int strips = std::max(1, (storage == LBMHD_FP32 ? 512 : 1024) / tiles_x);
  return std::min(kDiagRows, (g.ny + strips - 1) / strips);
}

static long long diag_units(int storage, const Geom& g) {
  const long long tiles_x = (g.nx + kDiagThreads - 1) / kDiagThreads;
  const int rows = diag_rows(storage, g);
  return tiles_x * ((g.ny + rows - 1) / rows);
}

int diag_partials(int storage, const Geom& g) {
  return int(std::min<long long>(kDiagBlocks, diag_units(storage, g)));
}

// A block to a row (k_diag_row; the strips above are then one row) while each has
// a CU of its own: us per interval of one step and its diagnostics, walking / by
// the row, FP32 64^2 16.7 / 12.5, 128^2 17.1 / 14.1, 256^2 18.7 / 17.5, 400^2 (800
// blocks) 28.9 / 29.0, 512^2 30.7 / 32.9.
bool diag_by_row(const Geom& g) {
  return (long long)((g.nx + kDiagThreads - 1) / kDiagThreads) * g.ny <= 256;
}

hipError_t launch_diag(int storage, const void* lat, double* part, double* out_dev,
                       const Geom& g, hipStream_t s) {
  const int tiles_x = (g.nx + kDiagThreads - 1) / kDiagThreads;
  const long long units = diag_units(storage, g);
  const int nparts = diag_partials(storage, g), rows = diag_rows(storage, g);
  if (diag_by_row(g))
    with_bools([&](auto fp32) {
      constexpr int ST = fp32() ? LBMHD_FP32 : LBMHD_FP16;
      hipLaunchKernelGGL((k_diag_row<ST, false, false>), dim3(nparts), dim3(kDiagRowThreads), 0, s,
                         static_cast<const typename Codec<ST>::T*>(lat), nullptr, part, g, Rates{},
                         tiles_x);
    }, storage == LBMHD_FP32);
  else if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_diag<LBMHD_FP32>, dim3(nparts), dim3(kDiagThreads), 0, s,
                       static_cast<const float*>(lat), part, g, tiles_x, int(units), rows);
  else
    hipLaunchKernelGGL(k_diag<LBMHD_FP16>, dim3(nparts), dim3(kDiagThreads), 0, s,
                       static_cast<const _Float16*>(lat), part, g, tiles_x, int(units), rows);
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(256), 0, s, part, nparts, out_dev);
  return hipGetLastError();
}

hipError_t launch_step_diag(int storage, bool les, const void* src, void* dst, double* part,
                            double* out_dev, const Geom& g, const Rates& r, hipStream_t s) {
  const int tiles_x = (g.nx + kDiagThreads - 1) / kDiagThreads;
  const long long units = diag_units(storage, g);
  const int nparts = diag_partials(storage, g), rows = diag_rows(storage, g);
  if (diag_by_row(g)) {
    with_bools([&](auto fp32, auto l) {
      constexpr int ST = fp32() ? LBMHD_FP32 : LBMHD_FP16;
      using T = typename Codec<ST>::T;
      hipLaunchKernelGGL((k_diag_row<ST, true, l()>), dim3(nparts), dim3(kDiagRowThreads), 0, s,
                         static_cast<const T*>(src), static_cast<T*>(dst), part, g, r, tiles_x);
    }, storage == LBMHD_FP32, les);
  } else {
    if (storage != LBMHD_FP32) return hipErrorInvalidValue;
    with_bools([&](auto l) {
      hipLaunchKernelGGL(k_step_diag<l()>, dim3(nparts), dim3(kDiagThreads), 0, s,
                         static_cast<const float*>(src), static_cast<float*>(dst), part, g, r,
                         tiles_x, int(units), rows);
    }, les);
  }
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(256), 0, s, part, nparts, out_dev);
  return hipGetLastError();
}

hipError_t launch_macro_box(int storage, const void* lat, int w, double* rho, double* ux,
                            double* uy, double* bx, double* by, const Geom& g, hipStream_t s) {
  const unsigned nb = blocks_for((long long)(g.nx / w) * (g.ny / w), 256);
  if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_macro_box<LBMHD_FP32>, dim3(nb), dim3(256), 0, s,
                       static_cast<const float*>(lat), w, rho, ux, uy, bx, by, g);
  else
    hipLaunchKernelGGL(k_macro_box<LBMHD_FP16>, dim3(nb), dim3(256), 0, s,
                       static_cast<const _Float16*>(lat), w, rho, ux, uy, bx, by, g);
  return hipGetLastError();
}

hipError_t launch_mismatch(int storage, const void* lat, const double* ux_t, const double* uy_t,
                           const double* bx_t, const double* by_t, double* part, double* out_dev,
                           const Geom& g, hipStream_t s) {
  const long long n = (long long)g.nx * g.ny;
  const int nparts = int(std::min<long long>(kDiagBlocks, blocks_for(n, 256)));
  if (storage == LBMHD_FP32)
    hipLaunchKernelGGL(k_mismatch<LBMHD_FP32>, dim3(nparts), dim3(256), 0, s,
                       static_cast<const float*>(lat), ux_t, uy_t, bx_t, by_t, part, g);
  else
    hipLaunchKernelGGL(k_mismatch<LBMHD_FP16>, dim3(nparts), dim3(256), 0, s,
                       static_cast<const _Float16*>(lat), ux_t, uy_t, bx_t, by_t, part, g);
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(kSumThreads), 0, s, part, (long long)nparts, out_dev);
  return hipGetLastError();
}

hipError_t launch_sum(const double* in, long long n, double* out_dev, hipStream_t s) {
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(kSumThreads), 0, s, in, n, out_dev);
  return hipGetLastError();
}

}  // namespace lbk
