// lbmhd_impl.h -- internal declarations shared by the kernels and the C ABI
// of the gfx950 lattice Boltzmann MHD library (not installed, not part of
// the public interface in include/lbmhd.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbmhd.h"

namespace lbk {

// Device layout of one lattice: 19 planes, each ny rows of `pitch` elements
// (pitch >= nx, a multiple of 256 bytes), plane stride `plane` elements.
struct Geom {
  int nx, ny;
  int pitch;
  long long plane;
};

// Collision constants, precomputed on the host in FP64 and rounded once.
struct Rates {
  float s3q;      // s_3 / 4 with s_3 = s_4 = 1 / tau0 (fixed-rate case)
  float s5q;      // s_5 / 12 (= s_6 / 12)
  float s7q;      // s_7 / 180
  float s8q;      // s_8 / 20
  float sm;       // s_m = 1 / tau_m0 (fixed-rate case)
  float tau0;     // 3 nu + 1/2
  float tau0sq;   // tau0^2
  float taum0;    // 3 eta + 1/2
  float taum0sq;  // tau_m0^2
  float cf;       // 18 C_S Delta^2
  float cm;       // 36 C_S Delta^2
  // the same constants scaled by powers of two (exact), as the forward
  // collision uses them: 1 / (4 tau) = 1 / (tau0d + sqrt(tau0dsq + cf4 Q / rho)),
  // 1 / tau_m = 1 / (taum0h + sqrt(taum0hsq + cmq |A|))
  float tau0d;    // 2 tau0
  float tau0dsq;  // 4 tau0^2
  float cf4;      // 4 cf
  float taum0h;   // tau_m0 / 2
  float taum0hsq; // tau_m0^2 / 4
  float cmq;      // cm / 4
  // cross-helicity closure: sqrt(tau) and sqrt(tau_m) are the largest roots
  // of t^3 - p t - q = 0 (p = tau0, tau_m0)
  float stau0;    // sqrt(tau0)
  float staum0;   // sqrt(tau_m0)
  float kv;       // (9/2) C_S Delta^2:  q_v = kv (|P| / (rho tau_m))^(1/2)
  float kb;       // 3 sqrt(3) C_S Delta^2:  q_b = -kb sgn(X) |X|^(1/2)
  float qclip;    // q_b below which the root lies under max(sqrt(1/2), sqrt(tau_m0/3))
};

// The strips of rows of a row-walking kernel: `rows` rows each, `grid` strips
// launched (with xcd the count rounded up to a multiple of eight, so that each
// XCD gets whole strips; a block past the last strip returns at once).
struct Strips {
  int rows, grid;
  bool xcd;
};

// The strips of `rows` rows each, in the order by XCDs (which lets neighbouring
// tiles share their edge lines in one L2) where at most `idle` in 64 of the
// launched ones lie past the lattice.
inline Strips strips_of(int rows, int ny, int idle = 8) {
  const int n = (ny + rows - 1) / rows, pad = (n + 7) / 8 * 8;
  const bool xcd = (pad - n) * 64 <= idle * pad;
  return Strips{rows, xcd ? pad : n, xcd};
}

// About `want` blocks, never more while strips of `lo` rows allow it: a few
// blocks over an even round leave some CUs a round of their own.  Strips
// taller than `hi` become `big` rows (many rounds; there idle strips cost more
// than the order by XCDs gives, 2% at 5990 x 3900).  ms per step, rows rounded
// down and plain order /
// this rule: k_step_t3 1448^2 0.0326 / 0.0272, 2500^2 0.089 / 0.070,
// 5000 x 3000 0.186 / 0.156; k_step_nb2 0.064 / 0.044, 0.166 / 0.110,
// 0.345 / 0.242; k_adj_step2 0.086 / 0.065, 0.251 / 0.175, 0.530 / 0.409;
// 2048^2 and 4096^2, which split evenly, as before.
// One strip of up to two thirds of `want` tiles, a block on most CUs and two on
// some, becomes `few` (us per step, one strip / four: k_step_t3 70000 x 33 38.9 /
// 32.4, 80000 x 100 108 / 95, k_step_nb2 184 / 145 and 186 / 157 at 100 rows,
// k_adj_step2 281 / 216; 100000 columns, 391 tiles, 109 / 111, 188 / 195, 295 / 302).
inline Strips split_rows(long long tiles_x, int ny, int want, int lo, int hi, int big,
                         int few = 4) {
  long long n = want / tiles_x;
  n = n >= 8 ? n / 8 * 8 : (n > 1 ? n : 1);
  long long rows = (ny + n - 1) / n;
  if (rows > hi) return strips_of(big, ny, 0);
  if (tiles_x > want / 2 && tiles_x <= want * 2 / 3) rows = (ny + few - 1) / few;
  return strips_of(int(rows < lo ? lo : rows), ny);
}

constexpr int kNPop = 19;
constexpr int kDiagSlots = 16;   // doubles per diagnostics partial
constexpr int kDiagBlocks = 4096; // partials in the workspace (one per reducing block)

// Forward step: dst = C(S(src)).
hipError_t launch_step(int storage, bool les, const void* src, void* dst, const Geom& g,
                       const Rates& r, hipStream_t s, bool kept = false);
// Whether the row-walking step kernels store past the caches (non-temporal).
bool stores_bypass(const Geom& g, size_t esize, bool kept = false);
// Two forward steps in one pass: dst = C(S(C(S(src)))), equal to two
// launch_step calls; with mid != nullptr the intermediate state C(S(src)) is
// stored there as well.  src, dst and mid must not overlap.
hipError_t launch_step2(int storage, bool les, const void* src, void* dst, void* mid,
                        const Geom& g, const Rates& r, hipStream_t s);
// Three forward steps in one pass, FP32 storage only: dst = (C S)^3 src,
// equal to three launch_step calls; with mid1, mid2 != nullptr the states
// after one and two steps are stored there too.  The buffers do not overlap.
hipError_t launch_step_t3(bool les, const void* src, void* dst, void* mid1, void* mid2,
                          const Geom& g, const Rates& r, hipStream_t s);
// Whether launch_step2 beats two launch_step calls on this lattice: it needs
// enough blocks to fill the chip (measured crossover: 1024^2 FP32, 2048^2 FP16).
bool step2_pays(int storage, const Geom& g);
// In-place step on one lattice (AA pattern): phase 0 takes the natural
// layout to the reversed one, phase 1 back; launch_unswap_aa turns a
// reversed layout into the natural one in place.
hipError_t launch_step_aa(int storage, bool les, int phase, void* lat, const Geom& g,
                          const Rates& r, hipStream_t s);
hipError_t launch_unswap_aa(int storage, void* lat, const Geom& g, hipStream_t s);
// k = 3 or 2 steps on one FP32 lattice in its natural layout, in one pass over
// it after the strips' and tiles' halos are copied to `halo`
// (inplace_halo_bytes, 256-byte aligned); equal to k launch_step calls.
hipError_t launch_inplace_steps(bool les, int k, void* lat, void* halo, const Geom& g,
                                const Rates& r, hipStream_t s);
// Whether launch_inplace_steps beats the AA steps on this lattice, and the
// bytes of its halo copies (0 where it does not or they outgrow a quarter of it).
bool inplace_rows_pay(const Geom& g);
size_t inplace_halo_bytes(const Geom& g);
// Forward step that needs the neighbours' rho, j, B (lattice gradients):
// the kinetic closure (kin: filtered equilibria, filter width delta) and/or
// the eddy closure `eddy` (0 none, 1 Smagorinsky, 2 cross-helicity).
hipError_t launch_step_nb(int storage, int eddy, bool kin, const void* src, void* dst,
                          const Geom& g, const Rates& r, double delta, hipStream_t s);
// Two such steps in one pass: dst = C(S(C(S(src)))), equal to two
// launch_step_nb calls bit for bit; with mid != nullptr the intermediate state
// is stored there as well.  src, dst and mid must not overlap.
hipError_t launch_step_nb2(int storage, int eddy, bool kin, const void* src, void* dst,
                           void* mid, const Geom& g, const Rates& r, double delta, hipStream_t s);
// Whether launch_step_nb2 beats two launch_step_nb calls on this lattice.
bool step_nb2_pays(const Geom& g);
// k steps in one launch, tile by tile in LDS: dst = (C S)^k src for any closure
// (eddy, kin as launch_step_nb; eddy 0 or 1 without kin the plain and the
// Smagorinsky-MHD update), equal to k single steps bit for bit.  k is at least
// one and at most 5 (3 with neighbour terms), or what tile_steps gives.  src
// and dst do not overlap.  keep > 0 (k then what tile_keep gives): dst takes
// every second state instead of the last, every state with neighbour terms,
// keep bytes apart (at least a lattice).
hipError_t launch_tile(int storage, int eddy, bool kin, const void* src, void* dst, int k,
                       const Geom& g, const Rates& r, double delta, hipStream_t s,
                       size_t keep = 0);
// The steps of a launch that keeps states, and whether that beats launches
// that keep one each.
int tile_keep(bool nb, const Geom& g);
bool tile_keep_pays(int storage, bool nb, const Geom& g);
// The steps of one launch where tiles are the faster way (eddy, kin as
// launch_tile), or 0 where the row-walking kernels are.
int tile_steps(int storage, int eddy, bool kin, const Geom& g);
// Whether launch_tile takes regions of 64 x 32 sites (closures without neighbour
// terms; keep: a launch that keeps states).
bool tile_wide(int storage, int k, bool keep, const Geom& g);
// Where tile_steps is not 0: whether tiles are also faster for only k steps (nb:
// closures with neighbour terms).
bool tile_short_pays(int storage, bool nb, int k, const Geom& g);
// Equilibrium initialisation from FP64 fields.
hipError_t launch_init(int storage, const double* rho, const double* ux, const double* uy,
                       const double* bx, const double* by, void* lat, const Geom& g,
                       hipStream_t s);
// Plain populations <-> encoded lattice.
hipError_t launch_decode(int storage, const void* lat, double* out, const Geom& g, hipStream_t s);
hipError_t launch_encode(int storage, const double* in, void* lat, const Geom& g, hipStream_t s);
// Macroscopic fields of an encoded lattice (no streaming).
hipError_t launch_macro(int storage, const void* lat, double* rho, double* ux, double* uy,
                        double* bx, double* by, const Geom& g, hipStream_t s);
// Byte copy (vector loads/stores) for checkpoints.
hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s);
// Diagnostics in one pass over the lattice: per-block partials (at most
// kDiagBlocks x kDiagSlots doubles at part) folded into out_dev[0 .. 12].
hipError_t launch_diag(int storage, const void* lat, double* part, double* out_dev,
                       const Geom& g, hipStream_t s);
// Whether launch_diag and launch_step_diag give each row a block.
bool diag_by_row(const Geom& g);
// One step src -> dst (the plain or the Smagorinsky-MHD update) fused with the
// diagnostics of dst, results as launch_diag's.  FP16 storage: where
// diag_by_row.
hipError_t launch_step_diag(int storage, bool les, const void* src, void* dst, double* part,
                            double* out_dev, const Geom& g, const Rates& r, hipStream_t s);
// Number of block partials launch_diag writes for this lattice (<= kDiagBlocks).
int diag_partials(int storage, const Geom& g);
// Rows of a strip of both passes.
int diag_rows(int storage, const Geom& g);

// Box-averaged macroscopic fields (w x w blocks).
hipError_t launch_macro_box(int storage, const void* lat, int w, double* rho, double* ux,
                            double* uy, double* bx, double* by, const Geom& g, hipStream_t s);
// Mismatch to target fields: per-block partials (at most kDiagBlocks doubles at part)
// folded into out_dev[0].
hipError_t launch_mismatch(int storage, const void* lat, const double* ux_t, const double* uy_t,
                           const double* bx_t, const double* by_t, double* part, double* out_dev,
                           const Geom& g, hipStream_t s);

// Adjoint.
hipError_t launch_adj_seed(int storage, const void* lat, float* lam, const Geom& g,
                           const Geom& ga, hipStream_t s);
hipError_t launch_adj_seed_mismatch(int storage, const void* lat, const double* ux_t,
                                    const double* uy_t, const double* bx_t, const double* by_t,
                                    double scale, float* lam, const Geom& g, const Geom& ga,
                                    hipStream_t s);
hipError_t launch_adj_step(int storage, bool les, const void* state, const float* lam_next,
                           float* lam_prev, double* acc, const Geom& g, const Geom& ga,
                           const Rates& r, double delta2, hipStream_t s);
int adj_step_blocks(const Geom& g);
// Two reverse steps in one pass: lam_prev = R_t(R_{t+1}(lam_next)) from the
// state x_t alone (x_{t+1} is recomputed on chip), equal to two
// launch_adj_step calls with the stored x_{t+1} and x_t; the closure-constant
// derivatives of both steps are added to acc (block slots b and
// adj_step_blocks(g) + b).  Closures that read no neighbours: les_fwd, the
// forward step takes the Smagorinsky-MHD collision (as launch_step's les);
// les, the reverse steps differentiate it (les_fwd implies les).
hipError_t launch_adj_step2(int storage, bool les_fwd, bool les, const void* state,
                            const float* lam_next, float* lam_prev, double* acc, const Geom& g,
                            const Geom& ga, const Rates& r, double delta2, hipStream_t s);
// Whether launch_adj_step2 takes tiles of 28 x 12 sites (below 40000 sites smaller
// ones may come first) and not strips of rows.
bool adj_tile_pays(int storage, const Geom& g);
// Whether a sweep over every state takes its steps in pairs: from 512 blocks of
// 8-row strips on (below, acc gains each step's block sums in the slots and
// order of single steps).
bool adj_step2_pays(const Geom& g);
// The same reverse step for the kinetic closure (les = 2, or 3 with the
// Smagorinsky-MHD closure): one walk over strips of rows, the gradient
// adjoints of the neighbours kept on chip.
hipError_t launch_adj_step_kin(int storage, bool les, const void* state, const float* lam_next,
                               float* lam_prev, double* acc, const Geom& g, const Geom& ga,
                               const Rates& r, double delta2, hipStream_t s);
hipError_t launch_sum(const double* in, long long n, double* out_dev, hipStream_t s);
hipError_t launch_adj_fields(const float* lam0, const double* rho0, const double* ux0,
                             const double* uy0, const double* bx0, const double* by0,
                             double* gux, double* guy, double* gbx, double* gby, const Geom& ga,
                             int nx, int ny, hipStream_t s);

}  // namespace lbk
