// Fused Taylor-4 step kernels (Sec. 4 Taylor propagator applied to the
// dynamics of Sec. 3), for R = 1 and local (window 0) face operators.
//
// The step U = sum_{k<=4} (dt L)^k / k! is evaluated as the product of its two
// real quadratic factors, the same polynomial with a different rounding order:
//   t = a1 z + b1 dt L z,  v  = z + dt L t,       z = (psi, f),
//   s = a2 v + b2 dt L v,  z' = v + dt L s.
// Each factor reads nothing but its own input, so a launch of two stages
// moves 2 c + r bytes per point, and two launches need no second state buffer.
//
// Sweep layout:
//   * a workgroup owns an output tile of one x chunk (the whole row up to 128
//     columns), TY rows in y and TZ planes in z, and loads one halo row/plane
//     per fused stage on each side;
//   * one wavefront per y row, two consecutive x columns per lane; rows are
//     published in LDS as [column parity][lane] for the y neighbours, the x
//     neighbours come by lane shifts;
//   * the workgroup marches z: when plane zi is loaded, stage k works on plane
//     zi - k with its input's below/centre planes in registers, the plane above
//     being the previous stage's fresh output; a factor's input at the plane
//     of its second stage is the oldest plane of the first stage's queue;
//   * tiles are numbered so that consecutive tiles share an XCD and its L2.
// fused2_kernel runs two of the four stages per launch (two launches per step,
// two-deep halos) and also carries the zeroth- and first-order conditions.
// The first-order auxiliary stages are formed at face points only: on the x
// faces and the y-face row by the two halo waves (which do no stencil work),
// through small LDS rings; on the z-face plane by the row waves from
// registers.  The face sources enter the stage outputs of the face points
// (whole rows on y and z faces, one column at each end of a row on x faces).
// A launch reads one buffer and writes another, since neighbouring tiles read
// halos that a tile overwrites.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "device_util.h"
#include "fused.h"

using abc::Geometry;
using namespace abc_dev;

namespace {

constexpr int kCols = 128;

template <typename T> struct cpx;
template <> struct cpx<double> { using t = double2; };
template <> struct cpx<float> { using t = float2; };

struct FusedArgs {
  int nx, ny, nz;
  int ntx, xw;  // x chunks and output columns per chunk (two-stage kernel)
  int nty, ntiles, tiles_per_xcd;
  int rev;  // tiles in reverse (tile_of)
  double diag, off;
  double coef[5];
  double sa1, sa2;  // one-pass sweep: base scales of stages 1 and 3 (factored form)
  double2 m0, b0, a0;
  int face_off[7];
  int has_V;
  long long bstride, fstride;  // one-pass sweep over orbitals: elements between orbitals' psi / aux arrays
};

// Tile of a workgroup.  Consecutive tiles share an XCD and its L2.  The second
// factor runs over the tiles in reverse (rev): where the state is larger than
// the last-level cache it starts at the end that the first one wrote last, which
// is still there: 256^3 c128 336 -> 320 us/step, c64 186 -> 175, 320^3 c128
// 637 -> 609; 128^3, all of it in the cache, stays at 33.6.  One-pass launches
// gain nothing from it (118 -> 118 at 256x256x128), and choosing the direction
// costs them 0.3 us at their start (128^3 c64, no condition 19.4 -> 19.75).
__device__ __forceinline__ int tile_of(int b, int ntiles, int per_xcd, int rev) {
  if (per_xcd) return (b & 7) * per_xcd + (rev ? per_xcd - 1 - (b >> 3) : b >> 3);
  return rev ? ntiles - 1 - b : b;
}

template <typename C>
__device__ __forceinline__ C czero() {
  C z;
  z.x = 0;
  z.y = 0;
  return z;
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Neighbouring lanes' values by DPP (no LDS traffic): lane i receives lane
// i - 1 (shr) or i + 1 (shl); lanes past the wave's ends receive zero.
__device__ __forceinline__ double dpp_shift(double v, bool right) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = (int)b, hi = (int)(b >> 32);
  const int l2 = right ? __builtin_amdgcn_update_dpp(0, lo, 0x138, 0xF, 0xF, true)
                       : __builtin_amdgcn_update_dpp(0, lo, 0x130, 0xF, 0xF, true);
  const int h2 = right ? __builtin_amdgcn_update_dpp(0, hi, 0x138, 0xF, 0xF, true)
                       : __builtin_amdgcn_update_dpp(0, hi, 0x130, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((long long)h2 << 32) | (unsigned)l2);
}
__device__ __forceinline__ float dpp_shift(float v, bool right) {
  const int b = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, right ? __builtin_amdgcn_update_dpp(0, b, 0x138, 0xF, 0xF, true)
                                         : __builtin_amdgcn_update_dpp(0, b, 0x130, 0xF, 0xF, true));
}
template <typename C>
__device__ __forceinline__ C dpp_shift_c(C v, bool right) {
  C o;
  o.x = dpp_shift(v.x, right);
  o.y = dpp_shift(v.y, right);
  return o;
}
// The same, with the lane past the wave's end (lane 0 for shr, 63 for shl)
// receiving `edge` instead of zero (its destination is left as it was).
__device__ __forceinline__ double dpp_shift_edge(double v, bool right, double edge) {
  const long long b = __builtin_bit_cast(long long, v), e = __builtin_bit_cast(long long, edge);
  const int lo = (int)b, hi = (int)(b >> 32), elo = (int)e, ehi = (int)(e >> 32);
  const int l2 = right ? __builtin_amdgcn_update_dpp(elo, lo, 0x138, 0xF, 0xF, false)
                       : __builtin_amdgcn_update_dpp(elo, lo, 0x130, 0xF, 0xF, false);
  const int h2 = right ? __builtin_amdgcn_update_dpp(ehi, hi, 0x138, 0xF, 0xF, false)
                       : __builtin_amdgcn_update_dpp(ehi, hi, 0x130, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((long long)h2 << 32) | (unsigned)l2);
}
__device__ __forceinline__ float dpp_shift_edge(float v, bool right, float edge) {
  const int b = __builtin_bit_cast(int, v), e = __builtin_bit_cast(int, edge);
  return __builtin_bit_cast(float, right ? __builtin_amdgcn_update_dpp(e, b, 0x138, 0xF, 0xF, false)
                                         : __builtin_amdgcn_update_dpp(e, b, 0x130, 0xF, 0xF, false));
}
template <typename C, typename T>
__device__ __forceinline__ C dpp_shift_edge_c(C v, bool right, T ex, T ey) {
  C o;
  o.x = dpp_shift_edge(v.x, right, ex);
  o.y = dpp_shift_edge(v.y, right, ey);
  return o;
}

// One quadratic factor of the step per launch, y = (1 + sA X + b X^2) in with
// X = dt L:
//   stage 1:  t = sA in + cA L in   (cA = b dt),
//   stage 2:  out = in + cB L t     (cB = dt).
// Tiles are TY = 8 rows by TZ planes (pick_depth) by one x chunk: the whole
// row when nx <= 128, else chunks of at most 124 output columns loaded with
// a two-column halo on each side (the chunk edges see zero neighbours, which
// only corrupts the halo columns, never an output).  12 waves.
//
// Horner form reads the step's initial state again in its second launch
// (3 c + r bytes per point there) and needs a third state buffer: 256^3
// without a condition, 186 + 255 us per step at 8 planes against 2 x 181.
constexpr int kTY2 = 8, kHalo2 = 2, kChunk = kCols - 2 * kHalo2;
// tile depth: a launch of `tiles` tiles takes ceil(tiles / kTileSlots) rounds
// of TZ + 2 kHalo2 planes each, and a tile's start (LDS cleared, face data and
// first planes fetched) costs about kTileStart planes.  The depth of least
// cost is within 4 % of the fastest measured one from 31^3 to 256^3 (first
// order c128, us per step: 31^3 16.9 with 2 planes, 33.5 with 8; 96^3 31.8 with
// 5, 40.2 with 8, 45.9 with 4; 128^3 45.0 with 8, 66 with 16; 160^3 122 with 16,
// 131 with 8)
constexpr int kTileSlots = 256, kTileStart = 2;

// one box of a (possibly batched) two-stage launch
struct Box2 {
  FusedArgs a;
  const void* in;
  void* out;
  const void* V;
  const double2* av;
  double2* aux_out;
  int tile_begin;  // first global tile of this box in the launch
  int pad;
};

// What a launch does beside the factor (the adjoint's needs): kKeep writes
// the stage-1 output t of its own points to `keep`; kGrad accumulates the
// gradient with respect to V (Grad2).
enum { kPlain = 0, kKeep = 1, kGrad = 2 };

// Gradient with respect to V of one factor, F = 1 + a X + b X^2 with X = dt L
// and dL/dV = -i: for the adjoint state l at the factor's output side, the
// forward factor's input y and stage-1 output t = a y + b X y, and the
// adjoint factor's own stage-1 output tau = a l + b X^H l,
//   gV += dt (Im(conj(l) t) + Im(conj(tau - a l) y)).
// The adjoint launch holds l and tau of its own points when it writes its
// output, so the gradient costs the reads of t and y and the update of gV
// instead of three kept adjoint stages and a pass of its own (first order,
// 96^3 x 48 steps with sqrt checkpoints: 8.6 to 5.9 ms with the depth rule).
// The increment tau - a l is taken as a difference.  Carried as stage 1 formed it
// instead: the same error but for a single step (80-bit reference, 14 x 15 x 16, dt
// 1e-2 to 1e-6; one step's probability 8.3e-17 -> 7.5e-17 of its terms) and 14 % of
// the time.
template <typename C>
struct Grad2 {
  const C* t;
  const C* y;
  double* gV;
  double dt;
};

template <typename T, int ORDER, int TZ, int MODE>
__device__ __forceinline__ void fused2_body(const typename cpx<T>::t* __restrict__ w_in,
                                            typename cpx<T>::t* __restrict__ out, const T* __restrict__ V,
                                            const FusedArgs& a, double sA, double cA, double cB,
                                            const double2* __restrict__ av, double2* __restrict__ aux_out, int tile,
                                            typename cpx<T>::t* __restrict__ keep,
                                            const Grad2<typename cpx<T>::t>& gr) {
  using C = typename cpx<T>::t;
  constexpr int TY = kTY2, H = kHalo2;
  constexpr int ROWS = TY + 2 * H;
  constexpr int NT = 64 * ROWS;
  constexpr int ITERS = TZ + 2 * H;
  constexpr bool FO = ORDER == 3;
  constexpr int FP = TZ + 2, FR = ROWS - 2;
  // first-order face data in LDS (sizes in double2; 1 = unused)
  constexpr int NXG = FO ? 2 * FP * FR : 1, NYG = FO ? FP * kCols : 1;
  constexpr int NVX = FO ? 2 * TY * 2 : 1, NVY = FO ? 2 * kCols : 1;
  // Rows published for the y neighbours (the x neighbours come by lane shifts): the stage-1 inputs w of every row
  // and the stage-1 outputs s1 of rows 1 .. ROWS-2 (the only rows stage 2
  // reads).  Double-buffered (one barrier per plane) when both buffers fit in
  // the 160 KiB of LDS beside the face data.
  constexpr int kPlaneBytes = (2 * ROWS - 2) * 2 * 64 * (int)sizeof(C);
  constexpr int kFaceBytes = 16 * (NXG + NYG + NVX + NVY);
  constexpr int DBN = 2 * kPlaneBytes + kFaceBytes <= 160 * 1024 ? 2 : 1;
  __shared__ C plw[DBN][ROWS][2][64];
  __shared__ C pls[DBN][ROWS - 2][2][64];

  const int lane = threadIdx.x & 63;
  const int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform row
  const int tx = tile % a.ntx, rest = tile / a.ntx;
  const int ty = rest % a.nty, tz = rest / a.nty;
  const int y0 = ty * TY, z0 = tz * TZ;
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int sz = nx * ny;
  const int y = y0 - H + r;
  const bool row_in = y >= 0 && y < ny;
  const int ybase = y * nx;
  const bool own_row = r >= H && r < H + TY && row_in;
  // columns: x = xb + 2 lane + c; owned outputs in [xo, xe)
  const int xo = tx * a.xw, xe = min(xo + a.xw, nx);
  const int xb = a.ntx == 1 ? 0 : xo - H;

  for (int i = threadIdx.x; i < DBN * ROWS * 2 * 64; i += NT) (&plw[0][0][0][0])[i] = czero<C>();
  for (int i = threadIdx.x; i < DBN * (ROWS - 2) * 2 * 64; i += NT) (&pls[0][0][0][0])[i] = czero<C>();

  C Yc[2][2], Yb[2][2];  // stage inputs: centre / below (j = 0: w, j = 1: stage-1 output)
  T Vd[2][2];            // V at planes zi-1, zi-2
  C pf[2];               // the next plane's fields
  T pv[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      Yc[j][c] = Yb[j][c] = czero<C>();
      Vd[j][c] = T(0);
    }
  }
  const T diag = T(a.diag), off = T(a.off);
  const unsigned cbytes = (unsigned)(nz * sz) * (unsigned)sizeof(C);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(w_in, cbytes);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(V, a.has_V ? (unsigned)(nz * sz) * (unsigned)sizeof(T) : 0u);

  // plane zz; cells outside the box read as zero
  auto fetch = [&](int zz) {
    const bool ok = row_in && zz >= 0 && zz < nz;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int x = xb + 2 * lane + c;
      const bool in = ok && x >= 0 && x < nx;
      const unsigned idx = in ? (unsigned)(zz * sz + ybase + x) : 0u;
      bload(rw, in ? idx * (unsigned)sizeof(C) : kOob, pf[c]);
      bload(rv, in ? idx * (unsigned)sizeof(T) : kOob, pv[c]);
    }
  };
  fetch(z0 - H);
  const T s1 = T(sA);
  T cfA[2], cfB[2];  // the stages' coefficients, zero for columns outside the box
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int x = xb + 2 * lane + c;
    const bool in = x >= 0 && x < nx;
    cfA[c] = in ? T(cA) : T(0);
    cfB[c] = in ? T(cB) : T(0);
  }
  // stage 1 runs on rows 1 .. ROWS-2, stage 2 on the tile's own rows
  const bool s1on = r >= 1 && r < ROWS - 1, s2on = r >= 2 && r < ROWS - 2;

  // First order: the tile's face data, read once before the sweep.
  //  * x faces (both sides), in LDS: the auxiliary input g = av over the
  //    stage-1 planes z0-1 .. z0+TZ and rows 1 .. ROWS-2 (the halo waves form
  //    v and the outputs).
  //  * the tile's z-face plane, if it has one (at most one when
  //    nz >= TZ + 2): each row wave holds g of its own row there in
  //    registers.
  //  * the tile's y-face row, if it has one (at most one when
  //    ny >= TY + 2), in LDS: g over the stage-1 planes.  The halo waves form
  //    its stage-2 source and auxiliary outputs during the sweep, as for the
  //    x faces.
  // The stage-2 source is v = sA g + cA (b g + a w) and the auxiliary output
  // g + cB (b v + a t).  Every thread issues all of its loads before using
  // any, so the staging costs one memory round trip, overlapped with the
  // first plane fetch.
  __shared__ double2 fxg[NXG];  // [side][plane][row]
  __shared__ double2 fyg[NYG];  // [plane][local column]
  // z face: g of this wave's row at the face plane, per column
  double2 gz[2] = {make_double2(0, 0), make_double2(0, 0)};
  // auxiliary stages v of the next two planes: x faces [plane & 1][own row]
  // [side], y-face row [plane & 1][local column]
  __shared__ double2 vx[NVX];
  __shared__ double2 vy[NVY];
  int yface = -1, zface = -1;  // face index (2/3, 4/5) of the tile's y row / z plane
  // face slab offsets as scalars (a per-lane index into the argument array
  // would make the compiler loop over the distinct indices)
  const int off_x0 = a.face_off[0], off_x1 = a.face_off[1];
  int off_y = 0, off_z = 0;
  if (FO) {
    const int ylo = y0 - H + 1, zlo = z0 - 1;
    if (ylo <= 0) yface = 2;
    else if (ylo <= ny - 1 && ny - 1 < ylo + FR) yface = 3;
    if (zlo <= 0) zface = 4;
    else if (zlo <= nz - 1 && nz - 1 < zlo + FP) zface = 5;
    off_y = yface == 3 ? a.face_off[3] : a.face_off[2];
    off_z = zface == 5 ? a.face_off[5] : a.face_off[4];
    constexpr int KX = (NXG + NT - 1) / NT, KYG = (NYG + NT - 1) / NT;
    double2 rx[KX], ryg[KYG];
    if (zface >= 0 && row_in && r >= 1 && r < ROWS - 1) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int xx = xb + 2 * lane + c;
        if (xx >= 0 && xx < nx) gz[c] = av[off_z + ybase + xx];
      }
    }
#pragma unroll
    for (int j = 0; j < KX; ++j) {
      const int i = threadIdx.x + j * NT;
      rx[j] = make_double2(0, 0);
      if (i < NXG) {
        const int rr = i % FR, pl = (i / FR) % FP, side = i / (FR * FP);
        const int yy = ylo + rr, zz = zlo + pl;
        if (yy >= 0 && yy < ny && zz >= 0 && zz < nz) rx[j] = av[(side ? off_x1 : off_x0) + zz * ny + yy];
      }
    }
#pragma unroll
    for (int j = 0; j < KYG; ++j) {
      const int i = threadIdx.x + j * NT;
      const int lx = i % kCols, pl = i / kCols;
      const int xx = xb + lx, zz = zlo + pl;
      ryg[j] = make_double2(0, 0);
      if (yface >= 0 && i < NYG && xx >= 0 && xx < nx && zz >= 0 && zz < nz) ryg[j] = av[off_y + zz * nx + xx];
    }
#pragma unroll
    for (int j = 0; j < KX; ++j) {
      const int i = threadIdx.x + j * NT;
      if (i < NXG) fxg[i] = rx[j];
    }
#pragma unroll
    for (int j = 0; j < KYG; ++j) {
      const int i = threadIdx.x + j * NT;
      if (i < NYG) fyg[i] = ryg[j];
    }
  }
  __syncthreads();

  // the y-face row when it is one of the tile's own rows (stage 2 and the
  // auxiliary outputs run there), as a tile row index; -1 otherwise
  int ryown = -1;
  if (FO && yface >= 0) {
    const int yf = yface == 3 ? ny - 1 : 0;
    if (yf >= y0 && yf < y0 + TY) ryown = yf - (y0 - H);
  }

#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int zi = z0 - H + it;
    // rows published by the previous iteration, and the buffers of the next
    auto& pw = plw[DBN == 2 ? (it & 1) : 0];
    auto& ps = pls[DBN == 2 ? (it & 1) : 0];
    auto& pwn = plw[DBN == 2 ? ((it + 1) & 1) : 0];
    auto& psn = pls[DBN == 2 ? ((it + 1) & 1) : 0];
    C prev[2];
    T vcur[2];
    C wm2[2], tau[2];  // the input and the stage-1 output at plane zi - 2 (before the slide)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      prev[c] = pf[c];
      vcur[c] = pv[c];
      wm2[c] = Yb[0][c];
      tau[c] = Yc[1][c];
    }
    if (it + 1 < ITERS) fetch(zi + 1);
    const int z2 = zi - 2;
    const bool own_out = own_row && it >= 2 * H && z2 < nz;
    // the gradient's operands at this iteration's output plane
    C gt[2], gy[2];
    double g0[2];
    if constexpr (MODE == kGrad) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int x = xb + 2 * lane + c;
        gt[c] = gy[c] = czero<C>();
        g0[c] = 0;
        if (own_out && x >= xo && x < xe) {
          const int idx = z2 * sz + ybase + x;
          gt[c] = gr.t[idx];
          gy[c] = gr.y[idx];
          g0[c] = gr.gV[idx];
        }
      }
    }
    // The halo waves' face work below runs after their prefetch is issued,
    // so that its latency overlaps the work.
    if (ORDER == 3 && (r == 0 || r == ROWS - 1) && lane < 2 * TY) {
      // First-order x faces, done by the two halo waves at the tile's edges
      // (idle in both stages), one lane per (own row, side).  They read the
      // rows published at the end of the previous iteration: pw holds w at
      // plane zi-1 and ps the stage-1 output s1 at plane zi-2.
      //  * top wave: v_f = sA g_f + cA (b g_f + a w) at plane zi-1, for the
      //    next iteration's stage 2 (LDS ring);
      //  * bottom wave: the auxiliary output g_f + cB (b v_f + a t) at
      //    plane zi-2 (v_f from the ring, written an iteration earlier).
      const int j = lane >> 1, side = lane & 1;
      const int rj = H + j, yj = y0 + j;
      const int xf = side ? nx - 1 : 0, lxf = xf - xb;
      if (lxf >= 0 && lxf < kCols && yj < ny) {
        const int ci = lxf & 1, li = lxf >> 1, rr = rj - 1;
        const int p1 = zi - 1, p2 = zi - 2;
        if (r == 0 && p1 >= z0 && p1 < z0 + TZ && p1 < nz) {
          const int pl = p1 - (z0 - 1);
          const double2 g = fxg[(side * FP + pl) * FR + rr];
          const C wv = pw[rj][ci][li];
          const double2 bg = cmul(a.b0, g), aw = cmul(a.a0, make_double2((double)wv.x, (double)wv.y));
          const double2 v = make_double2(sA * g.x + cA * (bg.x + aw.x), sA * g.y + cA * (bg.y + aw.y));
          vx[((p1 & 1) * TY + j) * 2 + side] = v;
        }
        if (r == ROWS - 1 && p2 >= z0 && p2 < z0 + TZ && p2 < nz && xf >= xo && xf < xe) {
          const double2 f0 = fxg[(side * FP + p2 - (z0 - 1)) * FR + rr];
          const double2 v = vx[((p2 & 1) * TY + j) * 2 + side];
          const C t1 = ps[rj - 1][ci][li];
          const double2 bv = cmul(a.b0, v), as1 = cmul(a.a0, make_double2((double)t1.x, (double)t1.y));
          aux_out[(side ? off_x1 : off_x0) + p2 * ny + yj] =
              make_double2(f0.x + cB * (bv.x + as1.x), f0.y + cB * (bv.y + as1.y));
        }
      }
    }
    if (ORDER == 3 && ryown >= 0 && (r == 0 || r == ROWS - 1)) {
      // The y-face row, by the same two halo waves over its whole width: the
      // top wave forms v = sA g + cA (b g + a w) at plane zi-1 into the ring;
      // the bottom wave writes the auxiliary output g + cB (b v + a t) at
      // plane zi-2.
      const int p = r == 0 ? zi - 1 : zi - 2;
      if (p >= z0 && p < z0 + TZ && p < nz) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int lx = 2 * lane + c, x = xb + lx;
          if (x < 0 || x >= nx) continue;
          const double2 g = fyg[(p - z0 + 1) * kCols + lx];
          if (r == 0) {
            const C wv = pw[ryown][c][lane];
            const double2 bg = cmul(a.b0, g), aw = cmul(a.a0, make_double2((double)wv.x, (double)wv.y));
            vy[(p & 1) * kCols + lx] = make_double2(sA * g.x + cA * (bg.x + aw.x), sA * g.y + cA * (bg.y + aw.y));
          } else if (x >= xo && x < xe) {
            const double2 v = vy[(p & 1) * kCols + lx];
            const C t1 = ps[ryown - 1][c][lane];
            const double2 bv = cmul(a.b0, v), as1 = cmul(a.a0, make_double2((double)t1.x, (double)t1.y));
            aux_out[off_y + p * nx + x] = make_double2(g.x + cB * (bv.x + as1.x), g.y + cB * (bv.y + as1.y));
          }
        }
      }
    }
    // First order: the x-face sources of this iteration's two stages, read
    // from LDS ahead of the stencil work so that their latency overlaps it.
    // Stage 1: av at plane zi-1; stage 2: v at plane zi-2 from the halo
    // wave's ring.  Every lane reads (the indices are clamped in range, and
    // do not bind in the active stages that use the values); only the lanes
    // holding a face column use them.  A branch here, or around the adds
    // below, splits the stage code into blocks that the compiler schedules
    // apart, which costs more than the extra reads and selects.
    // The y neighbours of both stages come from rows published by the previous
    // iteration; both columns' reads of a stage (without face data, of both
    // stages) are issued together, and a stage is one block for the scheduler.
    // With a branch per column each column's reads were waited for on their
    // own (160^3, us per step: first order 111 against 105, zeroth 90 against
    // 82, no condition 79 against 73).
    double2 gx[2] = {make_double2(0, 0), make_double2(0, 0)};
    int cxf = -1;
    C yn[2][2][2];  // [stage][column][below, above]
    auto read_rows = [&](int k) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        // stage 2: rows 1 and ROWS-2 read a neighbour that they will not use
        yn[k - 1][c][0] = k == 1 ? pw[r - 1][c][lane] : ps[max(r - 2, 0)][c][lane];
        yn[k - 1][c][1] = k == 1 ? pw[r + 1][c][lane] : ps[min(r, ROWS - 3)][c][lane];
      }
    };
    if (ORDER == 3) {
      const int x0 = xb + 2 * lane;
      cxf = (x0 == 0 || x0 == nx - 1) ? 0 : ((x0 + 1 == nx - 1) ? 1 : -1);
      const int side = x0 == 0 ? 0 : 1;
      const int rrc = min(max(r - 1, 0), FR - 1);
      const int plc = min(max(zi - z0, 0), FP - 1);
      const int jc = min(max(r - H, 0), TY - 1);
      gx[0] = fxg[(side * FP + plc) * FR + rrc];
      gx[1] = vx[(((zi - 2) & 1) * TY + jc) * 2 + side];
    }
    // stage k of this wave's row at plane zi - k, into o
    auto stage = [&](auto kc, const C* abv2, C* o) {
      constexpr int k = decltype(kc)::value;
      const int zk = zi - k;
      const double cf2 = k == 1 ? cA : cB;
      // x neighbours outside this lane's pair of columns (zero past the row's
      // ends; 32 LDS cycles a stage as reads of the published rows)
      const C xl = dpp_shift_c(Yc[k - 1][1], true), xr = dpp_shift_c(Yc[k - 1][0], false);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int x = xb + 2 * lane + c;
        const C cen = Yc[k - 1][c], bel = Yb[k - 1][c], abv = abv2[c];
        const C ym = yn[k - 1][c][0], yp = yn[k - 1][c][1];
        const C xm = c == 0 ? xl : Yc[k - 1][0];
        const C xp = c == 0 ? Yc[k - 1][1] : xr;
        // base: the factor's input, scaled in stage 1
        C b0 = wm2[c];
        if (k == 1) {
          b0.x = s1 * cen.x;
          b0.y = s1 * cen.y;
        }
        const T v = Vd[k - 1][c];
        T hr = (diag + v) * cen.x + off * (((bel.x + abv.x) + (ym.x + yp.x)) + (xm.x + xp.x));
        T hi = (diag + v) * cen.y + off * (((bel.y + abv.y) + (ym.y + yp.y)) + (xm.y + xp.y));
        if (ORDER == 2) {
          // zeroth-order local term nf m0 y, nf = number of faces at the
          // point (0 inside); computed for every lane without a branch, in
          // the stencil's precision
          const T nf = T((x == 0) + (x == nx - 1) + (y == 0) + (y == ny - 1) + (zk == 0) + (zk == nz - 1));
          const T m0x = T(a.m0.x), m0y = T(a.m0.y);
          hr += nf * (m0x * cen.x - m0y * cen.y);
          hi += nf * (m0x * cen.y + m0y * cen.x);
        }
        // columns outside the box stay zero (they are x neighbours): their
        // base is, and their coefficient
        const T cfc = k == 1 ? cfA[c] : cfB[c];
        o[c].x = b0.x + cfc * hi;
        o[c].y = b0.y - cfc * hr;
      }
      if constexpr (ORDER == 3) {
        // First order: the psi stage also sees -i sum_f g_f at face points,
        // with g = the auxiliary input (stage 1) or the auxiliary stage
        // v_f = sA g_f + cA (b g_f + a w) (stage 2), added to the plain stage
        // output as -i cf g.
        const int pl = zk - (z0 - 1);
        // x faces: at most one column per lane, its source read above,
        // added without a branch (zero for the other columns)
        {
          const double2 g = gx[k - 1];
          const bool c0 = cxf == 0, c1 = cxf == 1;
          if constexpr (std::is_same<T, double>::value) {
            o[0].x += cf2 * (c0 ? g.y : 0.0);
            o[0].y += -cf2 * (c0 ? g.x : 0.0);
            o[1].x += cf2 * (c1 ? g.y : 0.0);
            o[1].y += -cf2 * (c1 ? g.x : 0.0);
          } else {
            const T dx = T(cf2 * g.y), dy = T(-cf2 * g.x);
            o[0].x += c0 ? dx : T(0);
            o[0].y += c0 ? dy : T(0);
            o[1].x += c1 ? dx : T(0);
            o[1].y += c1 ? dy : T(0);
          }
        }
        // y and z faces: whole rows (wave-uniform), both columns of each lane,
        // sources precomputed at staging; stage 2 also writes the auxiliary
        // outputs Q + cB a s1 at owned points
        const bool fy = y == 0 || y == ny - 1, fz = zk == 0 || zk == nz - 1;
        if (fy || fz) {
          const bool own_pt = k == 2 && own_row && it >= 2 * H;
          const double2 ba = make_double2(cB * a.a0.x, cB * a.a0.y);
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const int lx = 2 * lane + c, x = xb + lx;
            if (x < 0 || x >= nx) continue;
            const bool own = own_pt && x >= xo && x < xe;
            double sr = 0, si = 0;
            double2 as1 = make_double2(0, 0);
            if (k == 2 && own) as1 = cmul(ba, make_double2((double)Yc[1][c].x, (double)Yc[1][c].y));
            // stage 1 adds g; stage 2 adds v = sA g + cA (b g + a w), w at this
            // plane, and at owned points writes g + cB b v + cB a t
            const double2 wv = make_double2((double)wm2[c].x, (double)wm2[c].y);
            auto face = [&](const double2 g, int oidx) {
              if (k == 1) {
                sr += g.x;
                si += g.y;
                return;
              }
              const double2 bg = cmul(a.b0, g), aw = cmul(a.a0, wv);
              const double2 v = make_double2(sA * g.x + cA * (bg.x + aw.x), sA * g.y + cA * (bg.y + aw.y));
              sr += v.x;
              si += v.y;
              if (own) {
                const double2 bv = cmul(a.b0, v);
                aux_out[oidx] = make_double2(g.x + cB * bv.x + as1.x, g.y + cB * bv.y + as1.y);
              }
            };
            if (fy) {
              // stage 1: g; stage 2: v from the halo wave's ring (the
              // auxiliary outputs are written there too)
              const double2 g = k == 1 ? fyg[pl * kCols + lx] : vy[(zk & 1) * kCols + lx];
              sr += g.x;
              si += g.y;
            }
            if (fz) face(gz[c], off_z + y * nx + x);
            o[c].x += T(cf2 * si);
            o[c].y += T(-cf2 * sr);
          }
        }
      }
      if constexpr (MODE == kKeep) {
        if (k == 1 && own_row && zk >= z0 && zk < z0 + TZ && zk < nz) {
          // the stage-1 output at the tile's own points
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const int x = xb + 2 * lane + c;
            if (x >= xo && x < xe) keep[zk * sz + ybase + x] = o[c];
          }
        }
      }
    };
    C o1[2], o2[2];
    o1[0] = o1[1] = o2[0] = o2[1] = czero<C>();
    if (it >= 2 && s1on) {
      const bool in1 = row_in && zi >= 1 && zi - 1 < nz, in2 = row_in && zi >= 2 && zi - 2 < nz;
      read_rows(1);
      if (!FO && it >= 4) read_rows(2);
      if (in1) stage(std::integral_constant<int, 1>(), prev, o1);
      if (it >= 4 && s2on && in2) {
        if (FO) read_rows(2);
        stage(std::integral_constant<int, 2>(), o1, o2);
      }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      Yb[0][c] = Yc[0][c];
      Yc[0][c] = prev[c];
      Yb[1][c] = Yc[1][c];
      Yc[1][c] = o1[c];
      prev[c] = o2[c];
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int x = xb + 2 * lane + c;
      if (own_out && x >= xo && x < xe) {
        out[z2 * sz + ybase + x] = prev[c];
        if constexpr (MODE == kGrad) {
          const double dx = tau[c].x - sA * wm2[c].x, dy = tau[c].y - sA * wm2[c].y;
          gr.gV[z2 * sz + ybase + x] =
              g0[c] + gr.dt * ((wm2[c].x * gt[c].y - wm2[c].y * gt[c].x) + (dx * gy[c].y - dy * gy[c].x));
        }
      }
      Vd[1][c] = Vd[0][c];
      Vd[0][c] = vcur[c];
    }
    // publish this plane's stage inputs; with a single buffer every wave
    // must first be done reading the previous ones
    if (DBN == 1) sync_lds();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      pwn[r][c][lane] = Yc[0][c];
      if (r >= 1 && r < ROWS - 1) psn[r - 1][c][lane] = Yc[1][c];
    }
    sync_lds();
  }
}

// one box, arguments in the kernel argument segment
template <typename T, int ORDER, int TZ, int MODE>
__global__ void __launch_bounds__(64 * (kTY2 + 2 * kHalo2)) fused2_kernel(
    const typename cpx<T>::t* __restrict__ in, typename cpx<T>::t* __restrict__ out, const T* __restrict__ V,
    FusedArgs a, double sA, double cA, double cB, const double2* __restrict__ av, double2* __restrict__ aux_out,
    typename cpx<T>::t* __restrict__ keep, Grad2<typename cpx<T>::t> gr) {
  const int tile = tile_of(blockIdx.x, a.ntiles, a.tiles_per_xcd, a.rev);
  fused2_body<T, ORDER, TZ, MODE>(in, out, V, a, sA, cA, cB, av, aux_out, tile, keep, gr);
}

// many boxes in one launch: the grid is the concatenation of the boxes' tiles
// (padded to a multiple of 8 for the XCD-aware order); each workgroup finds
// its box by binary search over the boxes' first tiles
template <typename T, int ORDER, int TZ>
__global__ void __launch_bounds__(64 * (kTY2 + 2 * kHalo2)) fused2_batch_kernel(
    const Box2* __restrict__ boxes, int nbox, int total_tiles, int half) {
  using C = typename cpx<T>::t;
  const int t = tile_of(blockIdx.x, total_tiles, gridDim.x >> 3, half);
  if (t >= total_tiles) return;
  int lo = 0, hi = nbox - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (boxes[mid].tile_begin <= t) lo = mid;
    else hi = mid - 1;
  }
  const Box2& b = boxes[lo];
  // coefficients of the box's own time step
  fused2_body<T, ORDER, TZ, kPlain>(static_cast<const C*>(b.in), static_cast<C*>(b.out), static_cast<const T*>(b.V),
                                    b.a, half ? b.a.sa2 : b.a.sa1, half ? b.a.coef[2] : b.a.coef[4], b.a.coef[1],
                                    b.av, b.aux_out, t - b.tile_begin, nullptr, Grad2<C>{});
}

// ---------------------------------------------------------------------------
// One-pass step: all four stages in one z-marching sweep, so the
// state, the potential and the result cross HBM once per step (40 B per
// point at complex128).  The tile is the whole row (nx <= 128) by TY rows by
// TZ planes, with four-deep halos in y and z; stage k is computed on rows
// k .. ROWS-1-k and planes z0-(4-k) .. z0+TZ+(3-k), so each stage is exact
// where the next reads it.  Register state per lane (two columns): the
// centre and below planes of each stage's input, the factor's base at the two
// oldest planes and V at the four stage planes.  The stage inputs' centre
// planes are published in LDS, level j (the output of stage j, level 0 =
// psi) only on the rows stage j+1 reads, double-buffered (one barrier per
// plane).  complex128: TY = 4, TZ = 16, 12 waves (about 160 VGPRs);
// complex64: TY = 8, TZ = 8, 16 or 24 (pick_depth4), 16 waves.
// ---------------------------------------------------------------------------
constexpr int kHalo4 = 4;
template <typename T> struct Tile4;
template <> struct Tile4<double> { static constexpr int TY = 4, TZ = 16; };
template <> struct Tile4<float> { static constexpr int TY = 8, TZ = 8; };  // TZ: 8, 16 or 24 (pick_depth4)

template <typename T>
__host__ __device__ constexpr int rows4() { return Tile4<T>::TY + 2 * kHalo4; }
// first LDS row of level j (level j holds the ROWS - 2j rows j .. ROWS-1-j)
template <typename T>
__host__ __device__ constexpr int level_base4(int j) { return j * rows4<T>() - j * (j - 1); }

// The step polynomial is applied as the product of its two real quadratic
// factors, P(x) = (1 + a1 x + b1 x^2)(1 + a2 x + b2 x^2), each in two stages
// (u = state, L = generator, D = dt):
//   stage 1: t = a1 u + b1 D L u      stage 2: v = u + D L t
//   stage 3: s = a2 v + b2 D L v      stage 4: u' = v + D L s
// The same polynomial as the Taylor sum, in another rounding order.  Every
// stage's base is its own input (stages 1, 3) or the input of the stage
// before it at the same plane (stages 2, 4), which the z queue already holds,
// so no separate copy of the step's initial state rides along.
// ORDER: 0 = zero outside the box, 2 = zeroth order (local face term),
// 3 = first order (Theorem 3.2, local face operators): the psi stage adds
// -i g_k sum_f A_f at face points (A_f the face's auxiliary stage input, g_k
// the stage's coefficient) and the auxiliary stage is base + g_k (b A + a
// psi_in), with the bases above.  A face point's auxiliary values pass
// through the four stages in four consecutive planes of the march:
//  * x faces and the tile's y-face row: helper waves (the halo rows, which
//    take part in no stage, and at a y face every row outside the box) run
//    the auxiliary stages one plane ahead of the row waves, from the stage
//    inputs published in LDS, and hand the next plane's sources A over
//    through LDS (double-buffered by plane parity); they keep the bases in
//    LDS slots indexed by plane & 3.  The jobs are split among the helpers
//    as described at the helper loop; the x faces' f0 is staged for the
//    whole march at the start, the y face's fetched a plane ahead;
//  * the z-face plane: one stage at a time is on it, so the row waves run
//    its auxiliary stage themselves (slots per thread; f0 read at stage 1).
// So the first-order tile needs ny > ROWS and nz > TZ + 4 (at most one face
// row and plane per tile), and with complex128 one plane buffer (two barriers
// per plane) to fit the slots in LDS.
// FULL: every lane's two columns lie in the box (nx == 128); otherwise the
// stage outputs of columns x >= nx are forced to zero (they are read as the
// x neighbours of the last column).
template <typename T, int ORDER, bool FULL, bool DB, int TZ>
__global__ void __launch_bounds__(64 * rows4<T>()) fused4_kernel(const typename cpx<T>::t* __restrict__ pin,
                                                                  typename cpx<T>::t* __restrict__ pout,
                                                                  const T* __restrict__ V, FusedArgs a,
                                                                  const double2* __restrict__ fin,
                                                                  double2* __restrict__ fout) {
  using C = typename cpx<T>::t;
  constexpr int TY = Tile4<T>::TY, H = kHalo4;
  constexpr int ROWS = rows4<T>();
  constexpr int NT = 64 * ROWS;
  constexpr int ITERS = TZ + 2 * H;
  constexpr int NLR = level_base4<T>(4);  // published rows over the four levels
  constexpr bool FO = ORDER == 3;
  // complex64: the z-face slots, which only their own thread reads, in
  // registers, and the 64 KB of LDS go to the second plane buffer (96^3 x 32
  // 532 -> 487 us/step); the x-face sources ready in the state's type (445 -> 428).
  // complex128 has neither the registers nor the LDS for these.  The sources as
  // FP32 neighbours against an FP64 product added to the stage's output: the x faces'
  // rms error against 64 bits is 0.73 of that one's over 60 boxes of 24^3 to 128^3, 1 to
  // 10 steps from zero auxiliary variables (whole state 1.00); one step from sources
  // that outweigh the state 3e4 times, 1.4
  constexpr bool ZREG = sizeof(T) == 4;
  constexpr bool XE = FO && sizeof(T) == 4;
  // rows as [column parity][lane] (x neighbours come by DPP, so no guard
  // cells); two buffers (DB: one barrier per plane) or one (two barriers)
  __shared__ C pl[DB ? 2 : 1][NLR][2][64];
  // first-order face data (sizes in double2; 1 when unused)
  constexpr int NXF = FO ? 2 * ROWS * ITERS : 1, NXS = FO ? 2 * 4 * 2 * ROWS : 1, NXB = FO ? 2 * ROWS * 4 : 1;
  constexpr int NYS = FO ? 2 * 4 * 2 * 64 : 1, NYB = FO ? 4 * 2 * 64 : 1, NZC = FO && !ZREG ? ROWS * 2 * 64 * 2 : 1;
  __shared__ double2 xf0[NXF];  // [march plane][side][row]        x-face f0
  __shared__ double2 xsrc[NXS];  // [plane parity][stage][side][row] x-face stage inputs A
  __shared__ C xe[XE ? NXS : 1];  // xsrc / off in the state's type (XE)
  __shared__ double2 xb[NXB];   // [plane & 3][side][row]          x-face bases
  __shared__ double2 ysrc[NYS];  // [plane parity][stage][c][lane]  y-face stage inputs A
  __shared__ double2 yb[NYB];   // [plane & 3][c][lane]            y-face bases
  __shared__ double2 zch[NZC];  // [row][c][A, base][lane]         z-face slots

  const int lane = threadIdx.x & 63;
  const int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform row
  // an orbital batch: blockIdx.y picks the orbital's arrays (V is shared)
  pin += (long long)blockIdx.y * a.bstride;
  pout += (long long)blockIdx.y * a.bstride;
  if (FO) {
    fin += (long long)blockIdx.y * a.fstride;
    fout += (long long)blockIdx.y * a.fstride;
  }
  int tile = blockIdx.x;
  if (a.tiles_per_xcd) tile = (blockIdx.x & 7) * a.tiles_per_xcd + (blockIdx.x >> 3);
  const int ty = tile % a.nty, tz = tile / a.nty;
  const int y0 = ty * TY, z0 = tz * TZ;
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int sz = nx * ny;
  const int y = y0 - H + r;
  const bool row_in = y >= 0 && y < ny;
  const int ybase = y * nx;
  const bool own_row = r >= H && r < H + TY && row_in;
  bool inx[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) inx[c] = FULL || 2 * lane + c < nx;

  for (int i = threadIdx.x; i < (DB ? 2 : 1) * NLR * 2 * 64; i += NT) (&pl[0][0][0][0])[i] = czero<C>();

  // first order: the faces the tile meets
  const int xh = nx - 1;  // high x-face column
  int yrow = -1, yface = -1;  // the tile row on a y face, and the face
  int zface_plane = -1, zface = -1;  // the z-face plane the march meets
  if (FO) {
    if (y0 - H <= 0) yrow = H - y0, yface = 2;
    else if (y0 - H + ROWS - 1 >= ny - 1) yrow = ny - 1 - (y0 - H), yface = 3;
    if (yrow < 1 || yrow > ROWS - 2) yrow = yface = -1;  // no stage runs on rows 0 and ROWS-1
    if (z0 - H <= 0) zface_plane = 0, zface = 4;
    else if (z0 + TZ + H - 1 >= nz - 1) zface_plane = nz - 1, zface = 5;
    // the x-face f0 over the march
    for (int i = threadIdx.x; i < NXF; i += NT) {
      const int q = i % ITERS, rr = (i / ITERS) % ROWS, side = i / (ITERS * ROWS);
      const int yy = y0 - H + rr, zz = z0 - H + q;
      double2 v = make_double2(0, 0);
      if (yy >= 0 && yy < ny && zz >= 0 && zz < nz) v = fin[a.face_off[side] + zz * ny + yy];
      xf0[(q * 2 + side) * ROWS + rr] = v;
    }
  }
  // Helper waves run in a loop of their own: the halo rows 0 and ROWS-1
  // (which take part in no stage) publish their psi row, and with the first
  // order every wave whose row lies outside the box (tiles at a y face) joins
  // them for the face jobs, the auxiliary stages of the plane's four stages:
  //  * without a y-face row (two helpers): helper 0 runs the x faces' stages
  //    1-2, helper 1 stages 3-4, one (stage, side, row) item per lane;
  //  * with one and at least five helpers: helpers 0-3 run the y-face row's
  //    stages 1-4 (two columns per lane), helper 4 all x-face items;
  //  * otherwise (a y-face row in a tile's halo, few helpers): helper 0 the
  //    stages 1-2 of both, the last helper stages 3-4.
  // Rows 0 and ROWS-1 also fetch the y face's f0 (even / odd columns).
  const int nlo = FO ? min(max(H - y0, 1), ROWS) : 1;            // rows 0 .. nlo-1
  const int hstart = FO ? min(max(ny - y0 + H, 0), ROWS - 1) : ROWS - 1;  // rows hstart ..
  const bool helper = r < nlo || r >= hstart;
  const int ycol = r == 0 ? 0 : 1;                     // f0 fetch of the y face
  const bool yfetch = FO && yrow >= 0 && (r == 0 || r == ROWS - 1) && 2 * lane + ycol < nx;

  C Yc[4][2], Yb[4][2];  // stage-k inputs (level k-1): centre / below plane
  T Dd[4][2];            // diagonal of H (stencil centre + V) at planes zi-1 .. zi-4
  C pf[2];               // psi and V of the next plane, fetched an iteration ahead
  T pv[2];
  double2 pfy;           // y-face job: the face's f0 at the next plane (the wave's column)
#pragma unroll
  for (int c = 0; c < 2; ++c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Yc[j][c] = Yb[j][c] = czero<C>();
      Dd[j][c] = T(0);
    }
  }
  pfy = make_double2(0, 0);
  const T diag = T(a.diag), off = T(a.off);
  const T sa1 = T(a.sa1), sa2 = T(a.sa2);
  const unsigned cbytes = (unsigned)(nz * sz) * (unsigned)sizeof(C);
  const __amdgpu_buffer_rsrc_t rp = make_rsrc(pin, cbytes);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(V, a.has_V ? (unsigned)(nz * sz) * (unsigned)sizeof(T) : 0u);
  const __amdgpu_buffer_rsrc_t rf = make_rsrc(fin, FO ? (unsigned)a.face_off[6] * 16u : 0u);
  // plane zz (and, for the y-face job, the face's f0 there); cells outside
  // the box read as zero (out-of-range offsets)
  auto fetch = [&](int zz, bool face_f0) __attribute__((always_inline)) {
    const bool ok = row_in && zz >= 0 && zz < nz;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const bool in = ok && inx[c];
      const unsigned idx = (unsigned)(zz * sz + ybase + 2 * lane + c);
      bload(rp, in ? idx * (unsigned)sizeof(C) : kOob, pf[c]);
      bload(rv, in ? idx * (unsigned)sizeof(T) : kOob, pv[c]);
    }
    if (FO && face_f0 && yfetch) {
      const bool okf = zz >= 0 && zz < nz;
      const unsigned fi = (unsigned)(a.face_off[yface] + zz * nx + 2 * lane + ycol);
      bload(rf, okf ? fi * 16u : kOob, pfy);
    }
  };
  fetch(z0 - H, true);
  __syncthreads();
  const double io = 1.0 / a.off;
  auto put_xe = [&](int i, double2 v) __attribute__((always_inline)) {
    xe[i].x = T(v.x * io);
    xe[i].y = T(v.y * io);
  };

  // one face point's auxiliary stage k: A its input, B the carried base,
  // ce the psi stage input there; returns the output and the next base
  auto aux_stage = [&](int k, double2 A, double2 B, double2 ce, double2& nB) __attribute__((always_inline)) {
    const double gk = a.coef[5 - k];
    const double2 bA = cmul(a.b0, A), ac = cmul(a.a0, ce);
    double2 base;
    if (k == 1 || k == 3) {
      const double sc = k == 1 ? a.sa1 : a.sa2;
      base = make_double2(sc * A.x, sc * A.y);
    } else {
      base = B;
    }
    const double2 nA = make_double2(base.x + gk * (bA.x + ac.x), base.y + gk * (bA.y + ac.y));
    nB = (k == 1 || k == 3) ? A : nA;  // f0 for stage 2, v for stage 4
    return nA;
  };

  if (helper) {
    const int nhelp = nlo + (ROWS - hstart);
    const int hid = r < nlo ? r : nlo + (r - hstart);
    // this helper's stages: x faces [xk0, xk1], the y-face row [yk0, yk1]
    int xk0 = 1, xk1 = 0, yk0 = 1, yk1 = 0;
    if (FO) {
      const bool yf = yrow >= 0;
      if (yf && nhelp >= 5) {
        if (hid < 4) yk0 = yk1 = hid + 1;
        else if (hid == 4) xk0 = 1, xk1 = 4;
      } else if (hid == 0) {
        xk0 = 1, xk1 = 2;
        if (yf) yk0 = 1, yk1 = 2;
      } else if (hid == nhelp - 1) {
        xk0 = 3, xk1 = 4;
        if (yf) yk0 = 3, yk1 = 4;
      }
    }
    const int nxi = (xk1 - xk0 + 1) * 2 * ROWS;  // x items of this helper
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int zi = z0 - H + it;
      const auto& rd = pl[DB ? (it & 1) : 0];
      auto& wr = pl[DB ? ((it + 1) & 1) : 0];
      const int par = it & 1, npar = (it + 1) & 1;
      C cur[2];          // psi of this row at plane zi (published below)
      const double2 fy = pfy;  // y-face f0 at plane zi (the next plane's stage 1)
#pragma unroll
      for (int c = 0; c < 2; ++c) cur[c] = pf[c];
      if (it + 1 < ITERS) fetch(zi + 1, true);
      if (FO) {
        // one item: the auxiliary stage k of a face point; loads first for
        // every item of a group, then the arithmetic and the stores (the
        // items are independent: each stage is at its own plane and slot)
        struct Item {
          double2 A, B, ce;
        };
        // x faces: item j = (stage xk0 + j / (2 ROWS), side, row), two rounds
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int jj = lane + 64 * q;
          if (jj < nxi) {
            const int k = xk0 + jj / (2 * ROWS), ch = jj % (2 * ROWS), side = ch / ROWS, row = ch % ROWS;
            const int zk = zi - k;
            const int yy = y0 - H + row;
            const int xcol = side ? xh : 0;
            const int lb = level_base4<T>(k - 1) - (k - 1);
            const int rr = min(max(row, k - 1), ROWS - k);  // a published row of level k-1
            const int bi = ((zk & 3) * 2 + side) * ROWS + row;
            const C ce = rd[lb + rr][xcol & 1][xcol >> 1];
            const Item in{xsrc[((par * 4 + (k - 1)) * 2 + side) * ROWS + row], xb[bi],
                          make_double2((double)ce.x, (double)ce.y)};
            const bool act = row >= k && row < ROWS - k && it >= 2 * k && yy >= 0 && yy < ny && zk >= 0 && zk < nz;
            if (act) {
              double2 nB;
              const double2 nA = aux_stage(k, in.A, in.B, in.ce, nB);
              if (k < 4) {
                xsrc[((npar * 4 + k) * 2 + side) * ROWS + row] = nA;
                if (XE) put_xe(((npar * 4 + k) * 2 + side) * ROWS + row, nA);
                xb[bi] = nB;
              } else if (row >= H && row < H + TY && zk >= z0 && zk < z0 + TZ) {
                fout[a.face_off[side] + zk * ny + yy] = nA;
              }
            }
            // the stage-1 input of the next plane (zi): f0
            if (k == 1) {
              const double2 f0 = xf0[(it * 2 + side) * ROWS + row];
              xsrc[((npar * 4 + 0) * 2 + side) * ROWS + row] = f0;
              if (XE) put_xe(((npar * 4 + 0) * 2 + side) * ROWS + row, f0);
            }
          }
        }
        // the y-face row: stages [yk0, yk1], both columns of the lane
        for (int k = yk0; k <= yk1; ++k) {
          const int zk = zi - k;
          const int lb = level_base4<T>(k - 1) - (k - 1);
          const int rr = min(max(yrow, k - 1), ROWS - k);
          Item in[2];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const C ce = rd[lb + rr][c][lane];
            in[c] = Item{ysrc[((par * 4 + (k - 1)) * 2 + c) * 64 + lane], yb[((zk & 3) * 2 + c) * 64 + lane],
                         make_double2((double)ce.x, (double)ce.y)};
          }
          const bool act = yrow >= k && yrow < ROWS - k && it >= 2 * k && zk >= 0 && zk < nz;
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            if (!act || !inx[c]) continue;
            double2 nB;
            const double2 nA = aux_stage(k, in[c].A, in[c].B, in[c].ce, nB);
            if (k < 4) {
              ysrc[((npar * 4 + k) * 2 + c) * 64 + lane] = nA;
              yb[((zk & 3) * 2 + c) * 64 + lane] = nB;
            } else if (yrow >= H && yrow < H + TY && zk >= z0 && zk < z0 + TZ) {
              fout[a.face_off[yface] + zk * nx + 2 * lane + c] = nA;
            }
          }
        }
        if (yfetch) ysrc[((npar * 4 + 0) * 2 + ycol) * 64 + lane] = fy;
      }
      if (!DB) sync_lds();
      if (r == 0 || r == ROWS - 1) {
#pragma unroll
        for (int c = 0; c < 2; ++c) wr[r == 0 ? 0 : level_base4<T>(1) - 1][c][lane] = cur[c];
      }
      sync_lds();
    }
    return;
  }

  double2 zA[2], zB[2];  // z-face slots (ZREG)
#pragma unroll
  for (int c = 0; c < 2; ++c) zA[c] = zB[c] = make_double2(0, 0);
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int zi = z0 - H + it;
    const auto& rd = pl[DB ? (it & 1) : 0];
    auto& wr = pl[DB ? ((it + 1) & 1) : 0];
    const int par = it & 1;
    C prev[2];   // the previous stage's output at the plane above (stage 1: psi(zi))
    T dcur[2];
    C ub[2];     // stage-2 base: psi at plane zi - 2
    C vb[2];     // stage-4 base: the stage-2 output at plane zi - 4
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      prev[c] = pf[c];
      dcur[c] = diag + pv[c];
      ub[c] = Yb[0][c];
      vb[c] = Yb[2][c];
    }
    if (it + 1 < ITERS) fetch(zi + 1, false);
#pragma unroll
    for (int k = 1; k <= 4; ++k) {
      const int zk = zi - k;
      const T cf = T(a.coef[5 - k]);
      const bool active = r >= k && r < ROWS - k && it >= 2 * k && row_in && zk >= 0 && zk < nz;
      C o[2];
      if (active) {
        // level k-1 rows r-1, r, r+1 (published at the end of the previous plane)
        const int lb = level_base4<T>(k - 1) - (k - 1);
        // First order: the x-face sources -i g A enter as the x neighbours
        // outside the box of the face columns, A / off: at the low face (and
        // at the high one on full rows) as the lane past the wave's end of the
        // DPP shift, else in place of the zero cell past the row's end.
        T e0x = T(0), e0y = T(0), e1x = T(0), e1y = T(0);
        if (XE) {
          const C s0 = xe[((par * 4 + (k - 1)) * 2 + 0) * ROWS + r];
          const C s1 = xe[((par * 4 + (k - 1)) * 2 + 1) * ROWS + r];
          e0x = s0.x, e0y = s0.y, e1x = s1.x, e1y = s1.y;
        } else if (FO) {
          const double2 s0 = xsrc[((par * 4 + (k - 1)) * 2 + 0) * ROWS + r];
          const double2 s1 = xsrc[((par * 4 + (k - 1)) * 2 + 1) * ROWS + r];
          e0x = T(s0.x * io), e0y = T(s0.y * io), e1x = T(s1.x * io), e1y = T(s1.y * io);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int x = 2 * lane + c;
          const C cen = Yc[k - 1][c], bel = Yb[k - 1][c], abv = prev[c];
          const C ym = rd[lb + r - 1][c][lane];
          const C yp = rd[lb + r + 1][c][lane];
          // x neighbours: the lane's other column, or the neighbouring lane's
          // (a row is one wave, so by DPP)
          C xm, xp;
          if (FO && !FULL) {
            // the high x face's neighbour: the cell past the row's end
            C q0 = Yc[k - 1][0], q1 = Yc[k - 1][1];
            if (c == 1 && 2 * lane == nx) q0.x = e1x, q0.y = e1y;
            if (c == 0 && 2 * lane + 1 == nx) q1.x = e1x, q1.y = e1y;
            xm = c == 0 ? dpp_shift_edge_c(Yc[k - 1][1], true, e0x, e0y) : Yc[k - 1][0];
            xp = c == 0 ? q1 : dpp_shift_c(q0, false);
          } else if (FO) {
            xm = c == 0 ? dpp_shift_edge_c(Yc[k - 1][1], true, e0x, e0y) : Yc[k - 1][0];
            xp = c == 0 ? Yc[k - 1][1] : dpp_shift_edge_c(Yc[k - 1][0], false, e1x, e1y);
          } else {
            xm = c == 0 ? dpp_shift_c(Yc[k - 1][1], true) : Yc[k - 1][0];
            xp = c == 0 ? Yc[k - 1][1] : dpp_shift_c(Yc[k - 1][0], false);
          }
          const T d = Dd[k - 1][c];
          T hr = d * cen.x + off * (((bel.x + abv.x) + (ym.x + yp.x)) + (xm.x + xp.x));
          T hi = d * cen.y + off * (((bel.y + abv.y) + (ym.y + yp.y)) + (xm.y + xp.y));
          if (ORDER == 2) {
            const T nf = T((x == 0) + (x == nx - 1) + (y == 0) + (y == ny - 1) + (zk == 0) + (zk == nz - 1));
            const T m0x = T(a.m0.x), m0y = T(a.m0.y);
            hr += nf * (m0x * cen.x - m0y * cen.y);
            hi += nf * (m0x * cen.y + m0y * cen.x);
          }
          if (k == 1 || k == 3) {
            const T sa = k == 1 ? sa1 : sa2;
            o[c].x = sa * cen.x + cf * hi;
            o[c].y = sa * cen.y - cf * hr;
          } else {
            const C b = k == 2 ? ub[c] : vb[c];
            o[c].x = b.x + cf * hi;
            o[c].y = b.y - cf * hr;
          }
        }
        if (FO) {
          // face sources -i g_k A_f, in FP64
          const double gk = a.coef[5 - k];
          // the tile's y-face row (whole wave)
          if (r == yrow) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              const double2 A = ysrc[((par * 4 + (k - 1)) * 2 + c) * 64 + lane];
              o[c].x += T(gk * A.y);
              o[c].y -= T(gk * A.x);
            }
          }
          // the z-face plane (wave-uniform: one stage at a time is on it)
          if (zk == zface_plane) {
            const bool own_pt = k == 4 && own_row && zk >= z0 && zk < z0 + TZ;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if (!inx[c]) continue;
              const C ce = Yc[k - 1][c];
              const int si = (r * 2 + c) * 128 + lane;  // A at si, base at si + 64
              const double2 A =
                  k == 1 ? fin[a.face_off[zface] + ybase + 2 * lane + c] : (ZREG ? zA[c] : zch[si]);
              const double2 B = k == 1 ? A : (ZREG ? zB[c] : zch[si + 64]);
              o[c].x += T(gk * A.y);
              o[c].y -= T(gk * A.x);
              double2 nB;
              const double2 nA = aux_stage(k, A, B, make_double2((double)ce.x, (double)ce.y), nB);
              if (k < 4) {
                if (ZREG) {
                  zA[c] = nA;
                  zB[c] = nB;
                } else {
                  zch[si] = nA;
                  zch[si + 64] = nB;
                }
              } else if (own_pt) {
                fout[a.face_off[zface] + ybase + 2 * lane + c] = nA;
              }
            }
          }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (!FULL && !inx[c]) o[c] = czero<C>();
      } else {
        o[0] = o[1] = czero<C>();
      }
      // stage k is the last reader of its input window: slide it
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        Yb[k - 1][c] = Yc[k - 1][c];
        Yc[k - 1][c] = prev[c];
        prev[c] = o[c];
      }
      // keep the next stage's LDS reads below this stage's arithmetic (with
      // all four stages' reads hoisted the registers run out)
      __builtin_amdgcn_sched_barrier(0);
    }
    // stage 4's output is the new state at plane zi - 4
    const int z4 = zi - 4;
    const bool own_out = own_row && it >= 2 * H && z4 < nz;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (own_out && inx[c]) pout[z4 * sz + ybase + 2 * lane + c] = prev[c];
      Dd[3][c] = Dd[2][c];
      Dd[2][c] = Dd[1][c];
      Dd[1][c] = Dd[0][c];
      Dd[0][c] = dcur[c];
    }
    // publish the next plane's stage inputs: level j on rows j .. ROWS-1-j
    // (with one buffer, after every wave is done reading it)
    if (!DB) sync_lds();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (r >= j && r < ROWS - j) {
        const int lr = level_base4<T>(j) + r - j;
#pragma unroll
        for (int c = 0; c < 2; ++c) wr[lr][c][lane] = Yc[j][c];
      }
    }
    sync_lds();
  }
}

// the step polynomial's factors: stage k reads coef[5 - k]
void set_factors(const abc_launch& L, FusedArgs& a) {
  a.coef[4] = L.fused_b1 * L.dt;
  a.coef[3] = L.dt;
  a.coef[2] = L.fused_b2 * L.dt;
  a.coef[1] = L.dt;
  a.coef[0] = 0;
  a.sa1 = L.fused_a1;
  a.sa2 = L.fused_a2;
}

// rounds of workgroups that a launch takes; over many rounds the partly
// filled last one hardly counts
double tile_rounds(long long tiles) {
  const double r = (double)tiles / kTileSlots;
  return r < 4 ? std::ceil(r) : r;
}

// planes per tile of the one-pass sweep for `count` boxes in a launch, and the
// plane iterations its workgroups take one after the other.  complex64: 8 planes
// give 128^3 its 256 tiles; many boxes fill the chip with 16 or 24 as well, which
// run through the 8 halo planes less often (us/step with 8, 16 and 24: 96^3 x 32
// first order 428, 357, 332, no condition 324, 256, 237; 48^3 x 32 first order
// 16 110, 24 99; 512 x 512 x 128 369, 304, 291)
struct Depth4 {
  int tz;
  double iters;
};
Depth4 pick_depth4(bool c64, int order, int ny, int nz, long long count) {
  const int ty = c64 ? Tile4<float>::TY : Tile4<double>::TY, tz0 = c64 ? Tile4<float>::TZ : Tile4<double>::TZ;
  Depth4 best{0, 0};
  for (int tz = tz0; tz <= (c64 ? 24 : 16); tz += 8) {
    if (tz > tz0 && order == ABC_FIRST && nz <= tz + kHalo4) break;  // one z face per tile
    const double it =
        tile_rounds(count * ((ny + ty - 1) / ty) * ((nz + tz - 1) / tz)) * (tz + 2 * kHalo4);
    if (!best.tz || it < best.iters) best = {tz, it};
  }
  return best;
}

template <typename T>
FusedArgs make_args4(const abc_launch& L, int tz) {
  FusedArgs a{};
  a.nx = L.g.nx;
  a.ny = L.g.ny;
  a.nz = L.g.nz;
  a.ntx = 1;
  a.xw = a.nx;
  a.nty = (a.ny + Tile4<T>::TY - 1) / Tile4<T>::TY;
  const int ntz = (a.nz + tz - 1) / tz;
  a.ntiles = a.nty * ntz;
  a.tiles_per_xcd = (a.ntiles % 8 == 0) ? a.ntiles / 8 : 0;
  const double s = 1.0 / (2.0 * L.h * L.h);
  a.diag = -3.0 * L.c[0] * s;
  a.off = -L.c[1] * s;
  set_factors(L, a);
  for (int f = 0; f < 7; ++f) a.face_off[f] = (int)L.g.face_off[f];
  a.m0 = L.fused_m0;
  a.b0 = L.fused_b0;
  a.a0 = L.a_loc[0];
  return a;
}

template <typename T>
FusedArgs make_args(const abc_launch& L) {
  FusedArgs a{};
  a.nx = L.g.nx;
  a.ny = L.g.ny;
  a.nz = L.g.nz;
  const int TY = kTY2, TZ = L.fused_tz;
  a.ntx = a.nx > kCols ? (a.nx + kChunk - 1) / kChunk : 1;
  a.xw = (a.nx + a.ntx - 1) / a.ntx;
  a.nty = (a.ny + TY - 1) / TY;
  const int ntz = (a.nz + TZ - 1) / TZ;
  a.ntiles = a.ntx * a.nty * ntz;
  a.tiles_per_xcd = (a.ntiles % 8 == 0) ? a.ntiles / 8 : 0;
  const double s = 1.0 / (2.0 * L.h * L.h);
  a.diag = -3.0 * L.c[0] * s;
  a.off = -L.c[1] * s;
  set_factors(L, a);
  for (int f = 0; f < 7; ++f) a.face_off[f] = (int)L.g.face_off[f];
  a.m0 = L.fused_m0;
  a.b0 = L.fused_b0;
  a.a0 = L.a_loc[0];
  return a;
}

// the tile depths the two-stage kernels are built for, and the kernel for one
constexpr int kDepths[] = {2, 3, 4, 5, 6, 8, 12, 16};

template <typename F>
hipError_t with_depth(int tz, F f) {
  switch (tz) {
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 5: f(std::integral_constant<int, 5>()); break;
    case 6: f(std::integral_constant<int, 6>()); break;
    case 8: f(std::integral_constant<int, 8>()); break;
    case 12: f(std::integral_constant<int, 12>()); break;
    case 16: f(std::integral_constant<int, 16>()); break;
    default: return hipErrorInvalidValue;
  }
  return hipSuccess;
}

// ORDER template argument of an order without periodic wrap
template <typename F>
hipError_t with_order(int order, F f) {
  switch (order) {
    case ABC_FIRST: return f(std::integral_constant<int, 3>());
    case ABC_ZEROTH: return f(std::integral_constant<int, 2>());
    default: return f(std::integral_constant<int, 0>());
  }
}

// one factor (half 0: the first, 1: the second) from (in, fin) to (out, fout)
template <typename T, int MODE>
hipError_t launch_factor(const abc_launch& L, FusedArgs a, int half, const typename cpx<T>::t* in,
                         typename cpx<T>::t* out, const double2* fin, double2* fout, const T* V,
                         typename cpx<T>::t* keep, Grad2<typename cpx<T>::t> gr, hipStream_t st, abc_timer* tm) {
  a.rev = half;
  const dim3 g(a.ntiles), b(64 * (kTY2 + 2 * kHalo2));
  const double sA = half ? a.sa2 : a.sa1, cA = half ? a.coef[2] : a.coef[4], cB = a.coef[1];
  const char* label = half ? "fused2_half_b" : "fused2_half_a";
  return with_order(L.order, [&](auto ord) {
    return with_depth(L.fused_tz, [&](auto tz) {
      abc_launch_kernel(tm, label, fused2_kernel<T, decltype(ord)::value, decltype(tz)::value, MODE>, g, b, st, in, out,
                        V, a, sA, cA, cB, fin, fout, keep, gr);
    });
  });
}

template <typename T>
hipError_t launch_factor_batch(int order, int tz, int half, const Box2* boxes, int nbox, int total, hipStream_t st,
                               abc_timer* tm) {
  const dim3 g((unsigned)((total + 7) / 8 * 8)), b(64 * (kTY2 + 2 * kHalo2));
  const char* label = half ? "fused2_batch_b" : "fused2_batch_a";
  return with_order(order, [&](auto ord) {
    return with_depth(tz, [&](auto d) {
      abc_launch_kernel(tm, label, fused2_batch_kernel<T, decltype(ord)::value, decltype(d)::value>, g, b, st, boxes,
                        nbox, total, half);
    });
  });
}

int max_depth(int order, int nz) {
  // first order: one z-face plane per tile needs nz >= TZ + 2
  return order == ABC_FIRST ? std::min(16, nz - 2) : 16;
}

}  // namespace

int fused_max_limit(int order, int nz) {
  const int m = max_depth(order, nz);
  return m >= 16 ? 16 : (m >= 8 ? 8 : 4);
}

namespace {

long long tiles2(const FusedBox& b, int tz) {
  const int ntx = b.nx > kCols ? (b.nx + kChunk - 1) / kChunk : 1;
  return (long long)b.count * ntx * ((b.ny + kTY2 - 1) / kTY2) * ((b.nz + tz - 1) / tz);
}

// Whether the one-pass sweep takes less time than two launches of two stages
// for one orbital in a box that both cover.  Either is estimated as rounds x
// planes marched x the time of a plane, the latter as measured at 128^3 and
// around it (us; the first order's one-pass sweep differs on partial rows):
//                    two-stage   one-pass
//   c128 first         1.45        1.65, 1.70 on rows under 128 columns
//   c128 zeroth        1.22        1.29
//   c128 no condition  1.12        1.15
//   c64  first         1.19        1.48, 1.39
//   c64  zeroth        0.88        1.20
//   c64  no condition  0.79        1.02
// and the two launches not faster than their 2 (2 c + r) bytes per point, at
// 5.2 TB/s while state, scratch and potential stay in the last-level cache
// (180 MB) and 4.6 TB/s beyond.  Measured (two-stage / one-pass, us per
// step): first order c128, 64 x 64 x 128 21.6 / 41.1, 128^3 40.8 / 43.0, 512 x
// 512 x 128 582 / 730; c64 96^3 25.9 / 25.0, 128^3 35.5 / 26.6; zeroth order c128, 96 x 96 x 128
// 25.7 / 32.3, 128^3 35.6 / 33.9, 256 x 256 x 128 145 / 128.
bool onepass_faster(const abc_params& p, const Geometry& g) {
  const bool c64 = p.dtype == ABC_C64, first = p.order == ABC_FIRST, full = p.nx == kCols;
  const int o = first ? 0 : (p.order == ABC_ZEROTH ? 1 : 2);
  constexpr double c2[2][3] = {{1.45, 1.22, 1.12}, {1.19, 0.88, 0.79}};
  constexpr double c4[2][3] = {{1.65, 1.29, 1.15}, {1.48, 1.20, 1.02}};
  const FusedBox b{p.nx, p.ny, p.nz, 1};
  const int tz = fused_pick_depth(p.order, 16, {b});
  const double n = (double)g.npts, csz = c64 ? 8 : 16;
  const double bytes = 2 * n * 2.5 * csz, rate = n * 2.5 * csz < 180e6 ? 5.2e6 : 4.6e6;
  const double est2 =
      std::max(2 * (tile_rounds(tiles2(b, tz)) * (tz + 2 * kHalo2) + kTileStart) * c2[c64][o], bytes / rate);
  const double it4 = pick_depth4(c64, p.order, p.ny, p.nz, 1).iters;
  const double est4 = (it4 + kTileStart) * c4[c64][o] * (first && !full ? (c64 ? 0.94 : 1.03) : 1.0);
  return est4 <= est2;
}

}  // namespace

int fused_pick_depth(int order, int limit, const std::vector<FusedBox>& boxes) {
  int best = 4;
  double best_cost = 0;
  bool any = false;
  for (int tz : kDepths) {
    bool ok = tz <= limit;
    long long tiles = 0;
    for (const FusedBox& b : boxes) {
      ok = ok && tz <= max_depth(order, b.nz);
      tiles += tiles2(b, tz);
    }
    if (!ok) continue;
    const double cost = tile_rounds(tiles) * (tz + 2 * kHalo2 + kTileStart);
    if (!any || cost < best_cost) {
      any = true;
      best = tz;
      best_cost = cost;
    }
  }
  return best;
}

int fused_tile_depth(const abc_launch& L, int orbitals) {
  if (L.fused_stages == 2) return L.fused_tz;
  return pick_depth4(L.dtype == ABC_C64, L.order, L.g.ny, L.g.nz, orbitals).tz;
}

bool fused_supported(const abc_params& p, std::string* why) {
  auto no = [&](const char* m) {
    if (why) *why = m;
    return false;
  };
  if (p.radius != 1) return no("radius 1 only");
  if (p.batch > 64) return no("at most 64 orbitals");
  if (p.order == ABC_PERIODIC) return no("periodic boxes use the staged path");
  if (p.order == ABC_SECOND) return no("the second order (box form) uses the staged path");
  if ((p.order == ABC_ZEROTH || p.order == ABC_FIRST) && (p.form != ABC_FORM_FACES || p.window != 0))
    return no("local (window 0) face operators only");
  if (p.nz < 5 || p.ny < 4 || p.nx < 4) return no("nx, ny >= 4 and nz >= 5");
  if (p.order == ABC_FIRST && (p.ny < kTY2 + 2 || p.nz < 6))
    return no("first order: ny >= 10 and nz >= 6 (one y-face row and one z-face plane per tile)");
  if ((long long)p.nx * p.ny * p.nz >= (1LL << 31)) return no("grid below 2^31 points");
  // raw buffer loads address each array with 32-bit byte offsets
  if ((long long)p.nx * p.ny * p.nz * (p.dtype == ABC_C64 ? 8 : 16) >= (1LL << 32) - 16)
    return no("state array below 4 GiB");
  return true;
}

bool fused_shell_case(const abc_params& p) {
  return p.order == ABC_FIRST && p.form == ABC_FORM_FACES && p.window > 0;
}

bool fused4_supported(const abc_params& p, std::string* why) {
  auto no = [&](const char* m) {
    if (why) *why = m;
    return false;
  };
  if (fused_shell_case(p)) {
    // the condition-free sweep plus the boundary-shell rounds: the sweep's
    // own limits, R = 1 and one orbital
    if (p.radius != 1) return no("one-pass sweep with a windowed face operator: radius 1 only");
    if (p.batch != 1 || p.meanfield != ABC_MF_NONE) return no("one-pass sweep: one orbital, no mean field");
    abc_params q = p;
    q.order = ABC_DIRICHLET;
    q.window = 0;
    return fused4_supported(q, why);
  }
  if (!fused_supported(p, why)) return false;
  if (p.nx > kCols) return no("one-pass sweep: nx <= 128");
  if (p.order == ABC_FIRST) {
    // at most one y-face row and one z-face plane per tile
    const bool c64 = p.dtype == ABC_C64;
    const int rows = c64 ? rows4<float>() : rows4<double>();
    const int tz = c64 ? Tile4<float>::TZ : Tile4<double>::TZ;
    if (p.ny <= rows || p.nz <= tz + kHalo4)
      return no("one-pass sweep, first order: ny > rows per tile and nz > planes per tile + 4");
  }
  return true;
}

// The Taylor-4 polynomial 1 + x + x^2/2 + x^3/6 + x^4/24 as the product of
// two real quadratics (1 + a1 x + b1 x^2)(1 + a2 x + b2 x^2): 24 P(x) =
// (x^2 + p x + q)(x^2 + (4 - p) x + 24/q) pairs its two conjugate root
// pairs, with (p, q) solving q + 24/q + p (4 - p) = 12 and
// 24 p / q + (4 - p) q = 24 (matching the x^2 and x coefficients; x^3 and
// x^0 hold by construction).  Newton's method from (3.5, 3.8); a_i = p_i/q_i,
// b_i = 1/q_i.  Returns false unless the product reproduces every
// coefficient to 1e-14.
bool taylor4_quadratic_factors(double* a1, double* b1, double* a2, double* b2) {
  double p = 3.5, q = 3.8;
  for (int it = 0; it < 50; ++it) {
    const double f1 = q + 24.0 / q + p * (4.0 - p) - 12.0;
    const double f2 = 24.0 * p / q + (4.0 - p) * q - 24.0;
    const double j11 = 4.0 - 2.0 * p, j12 = 1.0 - 24.0 / (q * q);
    const double j21 = 24.0 / q - q, j22 = -24.0 * p / (q * q) + (4.0 - p);
    const double det = j11 * j22 - j12 * j21;
    if (det == 0) return false;
    const double dp = (f1 * j22 - f2 * j12) / det, dq = (j11 * f2 - j21 * f1) / det;
    p -= dp;
    q -= dq;
    if (std::fabs(dp) + std::fabs(dq) < 1e-16 * (std::fabs(p) + std::fabs(q))) break;
  }
  const double p2 = 4.0 - p, q2 = 24.0 / q;
  *a1 = p / q;
  *b1 = 1.0 / q;
  *a2 = p2 / q2;
  *b2 = 1.0 / q2;
  // (1 + a1 x + b1 x^2)(1 + a2 x + b2 x^2) against 1, 1, 1/2, 1/6, 1/24
  const double c1 = *a1 + *a2, c2 = *b1 + *b2 + *a1 * *a2, c3 = *a1 * *b2 + *a2 * *b1, c4 = *b1 * *b2;
  return std::fabs(c1 - 1.0) < 1e-14 && std::fabs(c2 - 0.5) < 1e-14 && std::fabs(c3 - 1.0 / 6) < 1e-14 &&
         std::fabs(c4 - 1.0 / 24) < 1e-14;
}

abc_status fused_prepare(const abc_params& p, abc_launch& L, std::vector<void*>* allocs, size_t* bytes,
                         std::string& err) {
  // the one-pass sweep where it covers the parameters (automatic path) or
  // when asked for, else two launches of two stages per step, whose tile
  // depth the tuner may limit (4, 8 or 16 planes)
  L.fused_stages = 2;
  if (!taylor4_quadratic_factors(&L.fused_a1, &L.fused_b1, &L.fused_a2, &L.fused_b2)) {
    err = "fused path: factoring the Taylor polynomial failed";
    return ABC_EDEVICE;
  }
  // Automatic choice, one orbital: by the estimate of onepass_faster, up to
  // the largest state it was measured on (2.95 GB); beyond that the one-pass
  // sweep where it covers the parameters (first order: rows of 128 columns).
  // A windowed first-order operator takes the one-pass sweep with the
  // boundary-shell rounds only when asked for: at 128^3 it measured level
  // with the staged path, w = 8 145 against 141 us per step, exact sections
  // 182 against 185.
  // Orbital batches and the mean field (orbitals as boxes of one launch):
  // the one-pass sweep for complex64, two launches for complex128 (two launches
  // / one pass, us per step, first order: c64 24^3 x 2 17 / 25, 48^3 x 2 21 / 25, 32^3 x 8
  // 24 / 25, 48^3 x 8 46 / 40, 61^3 x 8 58 / 39, 96^3 x 32 496 / 321; c128 24^3 x 2 20 / 45,
  // 61^3 x 8 65 / 100, 96^3 x 32 620 / 803): small complex64 batches lose 5 to 8 us by it.
  const bool orbitals = p.batch > 1 || p.meanfield != ABC_MF_NONE;
  const bool large = (double)L.g.npts * (p.dtype == ABC_C64 ? 8 : 16) > 3e9;
  const bool auto4 = fused4_supported(p, nullptr) && !fused_shell_case(p) &&
                     (orbitals ? p.dtype == ABC_C64
                               : (large ? p.order != ABC_FIRST || p.nx == kCols : onepass_faster(p, L.g)));
  L.fused_shell = 0;
  if (p.path == ABC_PATH_ONEPASS || (p.path == ABC_PATH_AUTO && auto4)) {
    if (!fused4_supported(p, &err)) return ABC_ENOTSUP;
    L.fused_stages = 4;
    if (fused_shell_case(p)) {
      // four psi-sized and two face-aux buffers for the boundary-shell rounds
      L.fused_shell = 1;
      const size_t vb = (size_t)L.g.npts * (p.dtype == ABC_C64 ? 8 : 16);
      const size_t fb = (size_t)L.g.face_off[6] * sizeof(double2);
      for (int i = 0; i < 6; ++i) {
        void* ptr = nullptr;
        const size_t nb = i < 4 ? vb : fb;
        if (hipMalloc(&ptr, nb) != hipSuccess) {
          err = "one-pass sweep: boundary-shell buffers";
          return ABC_ENOMEM;
        }
        allocs->push_back(ptr);
        *bytes += nb;
        if (i < 4) L.shell.vol[i] = ptr;
        else L.shell.face[i - 4] = static_cast<double2*>(ptr);
      }
    }
  }
  L.fused_limit = fused_max_limit(p.order, p.nz);
  L.fused_tz = fused_pick_depth(p.order, L.fused_limit, {{p.nx, p.ny, p.nz, p.batch}});
  return ABC_OK;
}

namespace {

// One launch per step on the one-pass sweep; the ping-pong is arranged so
// that the last step writes the caller's buffers.
template <typename T, int ORDER>
void launch4(abc_timer* tm, bool full, dim3 g, dim3 b, hipStream_t st, const typename cpx<T>::t* src,
             typename cpx<T>::t* dst, const T* V, const FusedArgs& a, int tz, const double2* fin, double2* fout) {
  // first order, complex128: one plane buffer, so the face slots fit in LDS
  constexpr bool DB = ORDER != 3 || sizeof(T) == 4;
  auto launch = [&](auto kernel) { abc_launch_kernel(tm, "fused_step", kernel, g, b, st, src, dst, V, a, fin, fout); };
  constexpr int TZ = Tile4<T>::TZ;
  if constexpr (TZ < 16) {
    if (tz == 16) return launch(full ? fused4_kernel<T, ORDER, true, DB, 16> : fused4_kernel<T, ORDER, false, DB, 16>);
    if (tz == 24) return launch(full ? fused4_kernel<T, ORDER, true, DB, 24> : fused4_kernel<T, ORDER, false, DB, 24>);
  }
  launch(full ? fused4_kernel<T, ORDER, true, DB, TZ> : fused4_kernel<T, ORDER, false, DB, TZ>);
}

template <typename T>
hipError_t step4_t(const abc_launch& L, const abc_scratch& S, void* psi_v, double2* aux, const void* V_v, int n,
                   hipStream_t st, abc_timer* tm) {
  using C = typename cpx<T>::t;
  const int tz = pick_depth4(sizeof(T) == 4, L.order, L.g.ny, L.g.nz, 1).tz;
  FusedArgs a = make_args4<T>(L, tz);
  a.has_V = V_v != nullptr;
  C* user = static_cast<C*>(psi_v);
  C* scr = static_cast<C*>(S.y[0]);
  C* src = user;
  C* dst = scr;
  const bool first = L.order == ABC_FIRST;
  double2* fsrc = aux;
  double2* fdst = S.facc;
  if (n & 1) {
    hipError_t e = hipMemcpyAsync(scr, user, (size_t)L.g.npts * sizeof(C), hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && first)
      e = hipMemcpyAsync(S.facc, aux, (size_t)L.g.face_off[6] * sizeof(double2), hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
    src = scr;
    dst = user;
    fsrc = S.facc;
    fdst = aux;
  }
  const T* V = static_cast<const T*>(V_v);
  const dim3 g(a.ntiles), b(64 * rows4<T>());
  const bool full = a.nx == kCols;
  for (int s = 0; s < n; ++s) {
    if (L.fused_shell) {
      // the condition-free sweep, then the boundary-shell rounds (new aux,
      // the boundary's correction added to the swept state)
      launch4<T, 0>(tm, full, g, b, st, src, dst, V, a, tz, nullptr, nullptr);
      const hipError_t e = launch_shell_rounds(L, L.shell, src, V_v, fsrc, fdst, dst, st, tm);
      if (e != hipSuccess) return e;
    } else if (L.order == ABC_FIRST) launch4<T, 3>(tm, full, g, b, st, src, dst, V, a, tz, fsrc, fdst);
    else if (L.order == ABC_ZEROTH) launch4<T, 2>(tm, full, g, b, st, src, dst, V, a, tz, nullptr, nullptr);
    else launch4<T, 0>(tm, full, g, b, st, src, dst, V, a, tz, nullptr, nullptr);
    if (tm) tm->end_step();
    std::swap(src, dst);
    std::swap(fsrc, fdst);
  }
  return hipGetLastError();
}

// one step of B orbitals (arrays [B][npts], aux [B][nface]) on the one-pass
// sweep, one launch (blockIdx.y = orbital, V shared)
template <typename T>
hipError_t step4_orbitals(const abc_launch& L1, int B, const void* src, void* dst, const double2* fsrc, double2* fdst,
                          const void* V_v, hipStream_t st, abc_timer* tm) {
  using C = typename cpx<T>::t;
  const int tz = pick_depth4(sizeof(T) == 4, L1.order, L1.g.ny, L1.g.nz, B).tz;
  FusedArgs a = make_args4<T>(L1, tz);
  a.has_V = V_v != nullptr;
  a.bstride = L1.g.npts;
  a.fstride = L1.g.face_off[6];
  const dim3 g(a.ntiles, B), b(64 * rows4<T>());
  const bool full = a.nx == kCols;
  const C* s = static_cast<const C*>(src);
  C* d = static_cast<C*>(dst);
  const T* V = static_cast<const T*>(V_v);
  if (L1.order == ABC_FIRST) launch4<T, 3>(tm, full, g, b, st, s, d, V, a, tz, fsrc, fdst);
  else if (L1.order == ABC_ZEROTH) launch4<T, 2>(tm, full, g, b, st, s, d, V, a, tz, nullptr, nullptr);
  else launch4<T, 0>(tm, full, g, b, st, s, d, V, a, tz, nullptr, nullptr);
  return hipGetLastError();
}

template <typename T>
hipError_t step_t(const abc_launch& L, const abc_scratch& S, void* psi_v, double2* aux, const void* V_v, int n,
                  hipStream_t st, abc_timer* tm) {
  if (L.fused_stages == 4) return step4_t<T>(L, S, psi_v, aux, V_v, n, st, tm);
  using C = typename cpx<T>::t;
  FusedArgs a = make_args<T>(L);
  a.has_V = V_v != nullptr;
  C* psi = static_cast<C*>(psi_v);
  C* mid = static_cast<C*>(S.y[1]);
  double2* vmid = S.g[0];
  const T* V = static_cast<const T*>(V_v);
  // the state goes to the scratch and back: each factor reads only its input
  for (int s = 0; s < n; ++s) {
    hipError_t e = launch_factor<T, kPlain>(L, a, 0, psi, mid, aux, vmid, V, nullptr, {}, st, tm);
    if (e == hipSuccess) e = launch_factor<T, kPlain>(L, a, 1, mid, psi, vmid, aux, V, nullptr, {}, st, tm);
    if (e != hipSuccess) return e;
    if (tm) tm->end_step();
  }
  return hipGetLastError();
}

}  // namespace

// One step out of place, psi_in -> psi_mid -> psi_out: keep receives each
// factor's stage-1 output t.
hipError_t launch_step_fused_keep(const abc_launch& L, const abc_scratch& S, const double2* psi_in,
                                  const double2* aux_in, double2* psi_mid, double2* psi_out, double2* aux_out,
                                  const double* V, double2* const* keep, hipStream_t st) {
  if (L.dtype != ABC_C128) return hipErrorInvalidValue;
  FusedArgs a = make_args<double>(L);
  a.has_V = V != nullptr;
  hipError_t e = launch_factor<double, kKeep>(L, a, 0, psi_in, psi_mid, aux_in, S.g[0], V, keep[0], {}, st, nullptr);
  if (e == hipSuccess)
    e = launch_factor<double, kKeep>(L, a, 1, psi_mid, psi_out, S.g[0], aux_out, V, keep[1], {}, st, nullptr);
  return e == hipSuccess ? hipGetLastError() : e;
}

// One adjoint step of (lam, mu), in place through the scratch, adding the
// step's part of the gradient with respect to V to gV: La is the adjoint
// operator set, z, v and t the forward step's input, its state between the
// factors and the factors' stage-1 outputs, dt the forward time step.
hipError_t launch_step_fused_grad(const abc_launch& La, const abc_scratch& S, double2* lam, double2* mu,
                                  const double2* z, const double2* v, double2* const* t, const double* V, double* gV,
                                  double dt, hipStream_t st) {
  if (La.dtype != ABC_C128) return hipErrorInvalidValue;
  FusedArgs a = make_args<double>(La);
  a.has_V = V != nullptr;
  double2* mid = static_cast<double2*>(S.y[1]);
  hipError_t e = launch_factor<double, kGrad>(La, a, 1, lam, mid, mu, S.g[0], V, nullptr,
                                              Grad2<double2>{t[1], v, gV, dt}, st, nullptr);
  if (e == hipSuccess)
    e = launch_factor<double, kGrad>(La, a, 0, mid, lam, S.g[0], mu, V, nullptr, Grad2<double2>{t[0], z, gV, dt}, st,
                                     nullptr);
  return e == hipSuccess ? hipGetLastError() : e;
}

hipError_t launch_step_fused(const abc_launch& L, const abc_scratch& S, void* psi, double2* aux, const void* V,
                             int n_steps, hipStream_t st, abc_timer* tm) {
  if (L.dtype == ABC_C64) return step_t<float>(L, S, psi, aux, V, n_steps, st, tm);
  return step_t<double>(L, S, psi, aux, V, n_steps, st, tm);
}

// ---------------------------------------------------------------------------
// Batched boxes: one descriptor-driven launch per half-step for every group of
// boxes that share (order, precision, tile depth).
// ---------------------------------------------------------------------------

size_t fused_batch_desc_bytes(int nbox) { return (size_t)2 * nbox * sizeof(Box2); }

int fused_batch_build(const std::vector<FusedMember>& m, void* host) {
  const int nb = (int)m.size();
  Box2* hb = static_cast<Box2*>(host);
  int total = 0;
  for (int i = 0; i < nb; ++i) {
    const abc_launch& L = *m[i].L;
    const abc_scratch& S = *m[i].S;
    const bool first = L.order == ABC_FIRST;
    Box2& A = hb[i];
    Box2& B = hb[nb + i];
    A.a = L.dtype == ABC_C64 ? make_args<float>(L) : make_args<double>(L);
    A.a.has_V = m[i].V != nullptr;
    A.in = m[i].psi;
    A.out = S.y[1];
    A.V = m[i].V;
    A.av = first ? m[i].aux : nullptr;
    A.aux_out = first ? S.g[0] : nullptr;
    A.tile_begin = total;
    A.pad = 0;
    B = A;
    B.in = S.y[1];
    B.out = m[i].psi;
    B.av = first ? S.g[0] : nullptr;
    B.aux_out = first ? m[i].aux : nullptr;
    total += A.a.ntiles;
  }
  return total;
}

hipError_t launch_batch_fused(const std::vector<FusedMember>& m, int tz, const void* dev, int total, int n,
                              hipStream_t st, abc_timer* tm) {
  const int nb = (int)m.size();
  if (nb == 0 || n <= 0) return hipSuccess;
  const abc_launch& L0 = *m[0].L;
  // the descriptors' tile counts come from each box's depth; the kernels are
  // instantiated at tz, so every box must have been built at that depth
  for (int i = 0; i < nb; ++i)
    if (m[i].L->fused_tz != tz) return hipErrorInvalidValue;
  const Box2* db = static_cast<const Box2*>(dev);
  for (int s = 0; s < n; ++s) {
    for (int half = 0; half < 2; ++half) {
      const hipError_t e =
          L0.dtype == ABC_C64
              ? launch_factor_batch<float>(L0.order, tz, half, db + half * nb, nb, total, st, tm)
              : launch_factor_batch<double>(L0.order, tz, half, db + half * nb, nb, total, st, tm);
      if (e != hipSuccess) return e;
    }
    if (tm) tm->end_step();
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Orbital batches on the fused path
// ---------------------------------------------------------------------------
namespace {

// [n][B] <-> [B][n] through an LDS tile of 64 rows x B (B <= 64)
template <typename E>
__global__ void __launch_bounds__(256) aos_soa_kernel(const E* __restrict__ in, E* __restrict__ out, long long n,
                                                      int B, int to_soa) {
  extern __shared__ unsigned char smem[];
  E* tile = reinterpret_cast<E*>(smem);  // [B][65]
  const long long i0 = (long long)blockIdx.x * 64;
  const int cnt = (int)min((long long)64, n - i0);
  if (to_soa) {
    for (int t = threadIdx.x; t < cnt * B; t += blockDim.x) {
      const int i = t / B, b = t - i * B;
      tile[b * 65 + i] = in[(i0 + i) * B + b];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < 64 * B; t += blockDim.x) {
      const int b = t >> 6, i = t & 63;
      if (i < cnt) out[(long long)b * n + i0 + i] = tile[b * 65 + i];
    }
  } else {
    for (int t = threadIdx.x; t < 64 * B; t += blockDim.x) {
      const int b = t >> 6, i = t & 63;
      if (i < cnt) tile[b * 65 + i] = in[(long long)b * n + i0 + i];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < cnt * B; t += blockDim.x) {
      const int i = t / B, b = t - i * B;
      out[(i0 + i) * B + b] = tile[b * 65 + i];
    }
  }
}

template <typename E>
hipError_t transpose(const void* in, void* out, long long n, int B, bool to_soa, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + 63) / 64);
  aos_soa_kernel<E><<<blocks, 256, (size_t)B * 65 * sizeof(E), st>>>(static_cast<const E*>(in), static_cast<E*>(out),
                                                                      n, B, to_soa ? 1 : 0);
  return hipGetLastError();
}

// V + t0 rho + t3 rho^2 with rho = sum_b |psi_b|^2 (Sec. 4.3 mean field,
// simplified functional), from the orbital arrays of the current state
template <typename T>
__global__ void __launch_bounds__(256) meanfield_soa_kernel(const typename cpx<T>::t* __restrict__ cur,
                                                            const T* __restrict__ V, T* __restrict__ veff,
                                                            long long n, int B, T t0, T t3) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  T rho = 0;
  for (int b = 0; b < B; ++b) {
    const auto v = cur[(long long)b * n + p];
    rho += v.x * v.x + v.y * v.y;
  }
  const T base = V ? V[p] : T(0);
  veff[p] = base + t0 * rho + t3 * rho * rho;
}

}  // namespace

hipError_t launch_step_orbitals(OrbitalBatch& ob, void* psi, double2* aux, const void* V, int n, hipStream_t st,
                                abc_timer* tm) {
  if (n <= 0) return hipSuccess;
  const abc_launch& L1 = ob.L1;
  const int B = ob.B;
  const long long np = L1.g.npts, nf = L1.g.face_off[6];
  const bool c64 = L1.dtype == ABC_C64;
  const bool first = L1.order == ABC_FIRST;
  const size_t csz = c64 ? 8 : 16;
  // the result ends in array 0: the one-pass sweep alternates between the two
  // arrays (an odd count starts in array 1), the two-stage launches go to
  // array 1 and back
  const int in = (L1.fused_stages == 4 && (n & 1)) ? 1 : 0;
  hipError_t e = c64 ? transpose<float2>(psi, ob.soa[in], np, B, true, st)
                     : transpose<double2>(psi, ob.soa[in], np, B, true, st);
  if (e == hipSuccess && first) e = transpose<double2>(aux, ob.soa_f[in], nf, B, true, st);
  if (e != hipSuccess) return e;
  std::vector<FusedMember> m(B);
  for (int b = 0; b < B; ++b) {
    abc_scratch& S = ob.S[b];
    S.y[1] = static_cast<char*>(ob.soa[1]) + (size_t)b * np * csz;
    if (first) S.g[0] = ob.soa_f[1] + (size_t)b * nf;
    m[b] = {&L1, &S, static_cast<char*>(ob.soa[0]) + (size_t)b * np * csz, first ? ob.soa_f[0] + (size_t)b * nf : nullptr,
            ob.veff ? ob.veff : V};
  }
  if (L1.fused_stages == 4) {
    // one-pass sweep over all orbitals in one launch per step (blockIdx.y =
    // orbital); the ping-pong between arrays A and B ends in A
    for (int s = 0; s < n; ++s) {
      const int cur = (s & 1) == 0 ? in : 1 - in;
      if (ob.veff) {
        const void* cs = ob.soa[cur];
        const unsigned blocks = (unsigned)((np + 255) / 256);
        if (L1.meanfield == ABC_MF_SKYRME)
          e = skyrme_veff(*L1.pot, cs, true, B, c64, V, ob.veff, L1.t0, L1.t3, st, tm);
        else if (c64)
          abc_launch_kernel(tm, "meanfield", meanfield_soa_kernel<float>, dim3(blocks), dim3(256), st,
                            static_cast<const float2*>(cs), static_cast<const float*>(V),
                            static_cast<float*>(ob.veff), np, B, float(L1.t0), float(L1.t3));
        else
          abc_launch_kernel(tm, "meanfield", meanfield_soa_kernel<double>, dim3(blocks), dim3(256), st,
                            static_cast<const double2*>(cs), static_cast<const double*>(V),
                            static_cast<double*>(ob.veff), np, B, L1.t0, L1.t3);
        if (e != hipSuccess) return e;
      }
      const void* Vs = ob.veff ? ob.veff : V;
      e = c64 ? step4_orbitals<float>(L1, B, ob.soa[cur], ob.soa[1 - cur], first ? ob.soa_f[cur] : nullptr,
                                      first ? ob.soa_f[1 - cur] : nullptr, Vs, st, tm)
              : step4_orbitals<double>(L1, B, ob.soa[cur], ob.soa[1 - cur], first ? ob.soa_f[cur] : nullptr,
                                       first ? ob.soa_f[1 - cur] : nullptr, Vs, st, tm);
      if (e != hipSuccess) return e;
      if (tm) tm->end_step();
    }
    e = c64 ? transpose<float2>(ob.soa[0], psi, np, B, false, st) : transpose<double2>(ob.soa[0], psi, np, B, false, st);
    if (e == hipSuccess && first) e = transpose<double2>(ob.soa_f[0], aux, nf, B, false, st);
    return e;
  }
  const int par = n & 1;
  const size_t dbytes = fused_batch_desc_bytes(B);
  const void* vkey = ob.veff ? ob.veff : V;
  const void* ddev = static_cast<char*>(ob.desc_dev) + par * dbytes;
  if (!ob.desc_ok[par] || ob.desc_V[par] != vkey) {
    // a new descriptor set: never inside a graph capture (the copy would
    // read host memory that a later call may rewrite)
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone)
      return hipErrorStreamCaptureUnsupported;
    if (ob.pending && hipEventSynchronize(ob.copied) != hipSuccess) return hipErrorUnknown;
    void* dhost = static_cast<char*>(ob.desc_host) + par * dbytes;
    ob.desc_total = fused_batch_build(m, dhost);
    e = hipMemcpyAsync(const_cast<void*>(ddev), dhost, dbytes, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipEventRecord(ob.copied, st);
    if (e != hipSuccess) return e;
    ob.pending = true;
    ob.desc_V[par] = vkey;
    ob.desc_ok[par] = true;
  }
  const int total = ob.desc_total;
  for (int s = 0; s < n; ++s) {
    if (ob.veff) {
      const void* cur = ob.soa[0];
      const unsigned blocks = (unsigned)((np + 255) / 256);
      if (L1.meanfield == ABC_MF_SKYRME)
        e = skyrme_veff(*L1.pot, cur, true, B, c64, V, ob.veff, L1.t0, L1.t3, st, tm);
      else if (c64)
        abc_launch_kernel(tm, "meanfield", meanfield_soa_kernel<float>, dim3(blocks), dim3(256), st,
                          static_cast<const float2*>(cur), static_cast<const float*>(V), static_cast<float*>(ob.veff),
                          np, B, float(L1.t0), float(L1.t3));
      else
        abc_launch_kernel(tm, "meanfield", meanfield_soa_kernel<double>, dim3(blocks), dim3(256), st,
                          static_cast<const double2*>(cur), static_cast<const double*>(V),
                          static_cast<double*>(ob.veff), np, B, L1.t0, L1.t3);
      if (e != hipSuccess) return e;
    }
    const Box2* db = static_cast<const Box2*>(ddev);
    for (int half = 0; half < 2 && e == hipSuccess; ++half)
      e = c64 ? launch_factor_batch<float>(L1.order, ob.tz, half, db + half * B, B, total, st, tm)
              : launch_factor_batch<double>(L1.order, ob.tz, half, db + half * B, B, total, st, tm);
    if (e != hipSuccess) return e;
    if (tm) tm->end_step();
  }
  e = c64 ? transpose<float2>(ob.soa[0], psi, np, B, false, st) : transpose<double2>(ob.soa[0], psi, np, B, false, st);
  if (e == hipSuccess && first) e = transpose<double2>(ob.soa_f[0], aux, nf, B, false, st);
  return e;
}
