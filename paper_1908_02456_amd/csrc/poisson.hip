// Long-range TDHF potentials (Sec. 4.3): the Yukawa and Coulomb fields of the
// density rho = sum_j |phi_j|^2 from the Helmholtz and Poisson problems
//
//   (-Delta_h + 1/a^2) W_Y = 4 pi V0 a rho,      -Delta_h W_C = 2 pi e^2 rho,
//
// on the box with the wavefunctions' Laplacian of half-width R and zero
// values outside, solved every step by preconditioned conjugate gradients
// (the paper's method for these problems), FP64 throughout.  The two problems
// are independent systems solved side by side: every kernel takes both, one
// per blockIdx.y (a field that has converged returns at once).
//
// Preconditioner: the R = 1 operator -Delta_h + mu^2 with zero values outside
// is diagonalised by the sine transform (DST-I) along each axis, so its
// inverse is three dense n x n transforms, a division by its eigenvalues
// sum_a (2 - 2 cos(pi k_a / (n_a + 1))) / h^2 + mu^2, and three transforms
// back.  It is the exact inverse for R = 1, where CG stops after one
// iteration, and spectrally equivalent to the R = 2, 3 operators.  The
// transforms run on the FP64 matrix cores in three launches: the x and y
// transforms of a z-plane held in LDS, the z transform, division and z
// transform back of 16 columns, and the planes again, where the plane kernels
// also settle the start of the solve and form r.z.  A plane too large for LDS
// takes rocBLAS GEMMs, one per axis and direction.
//
// CG kernels run over a fixed grid of workgroups; every workgroup reduces
// the block partials in the same fixed order (alpha and beta are identical
// everywhere).  Solves start from the previous step's potential unless that
// start is worse than zero.  Convergence is decided right after the update of
// x and r, before the next preconditioner.  Either the host reads the flags
// after each iteration and stops at convergence, or (fixed mode) every solve
// issues a fixed number of iterations whose kernels return at once after
// convergence, with no host read, so that a step can be captured in a graph.
// Each solve's iteration count and whether it converged are added up on the
// device.
//
// 61^3, 8 orbitals, both fields, R = 1: 104 us per mean-field evaluation in 9
// launches and one wait (planes 13, columns 11, planes back 12.5, start and
// density 13, A p 6, x and r 9.4, check and potential 4 each); 446 with one field
// after the other, seven GEMM and scale launches per preconditioner, the
// preconditioner applied once more before convergence was looked at, and four
// waits.  96^3, 4 orbitals: 197 against 595; 130 x 140 x 80 (rocBLAS): 350
// against 789.  Of the planes' 13 us the products take 3.4 (122 planes leave
// half of the compute units idle); the matrix operand of the first 64 k loaded
// ahead of the barrier made them slower (15).
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <chrono>
#include <cmath>

#include "abc_internal.h"

namespace {

constexpr int kT = 256;
constexpr int kPT = 1024;  // threads of the plane transforms: one 16 x 16 tile per wave at 64 x 64

// scalar slots of a field in PotentialSolver::scal
enum { kRZ = 0, kBB = 1, kDone = 2, kIter = 3, kScal = 8 };
// bits of a flag not yet written (no double that a kernel stores)
constexpr long long kPending = -1;

struct Op {
  int nx, ny, nz;
  long long n;
  double diag[2];              // -3 c0 / h^2 + mu^2 per field
  double off[abc::kMaxR + 1];  // -c_k / h^2
};

// the fields solved together
struct Fields {
  int n;
  double mu2[2], scale[2];
  double* x[2];
};

template <int R>
__device__ __forceinline__ double apply_op(const Op& op, int f, const double* __restrict__ x, long long e) {
  const unsigned ue = (unsigned)e, row = ue / (unsigned)op.nx;  // n < 2^32 (its vectors fit the device)
  const int ix = (int)(ue - row * (unsigned)op.nx);
  const int iz = (int)(row / (unsigned)op.ny);
  const int iy = (int)(row - (unsigned)iz * (unsigned)op.ny);
  const long long sy = op.nx, sz = (long long)op.nx * op.ny;
  double acc = op.diag[f] * x[e];
#pragma unroll
  for (int k = 1; k <= R; ++k) {
    double s = 0;
    if (ix + k < op.nx) s += x[e + k];
    if (ix - k >= 0) s += x[e - k];
    if (iy + k < op.ny) s += x[e + k * sy];
    if (iy - k >= 0) s += x[e - k * sy];
    if (iz + k < op.nz) s += x[e + k * sz];
    if (iz - k >= 0) s += x[e - k * sz];
    acc += op.off[k] * s;
  }
  return acc;
}

// sum over the workgroup, the same value in every thread: lanes by halves,
// then the waves in order
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = sh[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) r += sh[w];
  __syncthreads();
  return r;
}

// sum of n partials in a fixed order (every workgroup gets the same value)
template <int NT>
__device__ __forceinline__ double sum_partials(const double* __restrict__ part, int n, double* sh) {
  double a = 0;
  for (int i = threadIdx.x; i < n; i += NT) a += part[i];
  return block_sum<NT>(a, sh);
}

// The partial sums of a field: r.r, b.b (start), p.q, r.z, `np` doubles each
struct Parts {
  double* base;
  int np;
  __device__ double* rr(int f) const { return base + (4 * f + 0) * (long long)np; }
  __device__ double* bb(int f) const { return base + (4 * f + 1) * (long long)np; }
  __device__ double* pq(int f) const { return base + (4 * f + 2) * (long long)np; }
  __device__ double* rz(int f) const { return base + (4 * f + 3) * (long long)np; }
};

// density, and per field b = scale rho, r = b - A x, partials of r.r and b.b
template <typename C, int R>
__global__ void __launch_bounds__(kT) cg_init_kernel(Op op, const C* __restrict__ psi, int B, int soa,
                                                     double* __restrict__ rho, Fields fs, double* __restrict__ r,
                                                     Parts part) {
  __shared__ double sh[kT / 64];
  double rr[2] = {0, 0}, bb[2] = {0, 0};
  for (long long e = (long long)blockIdx.x * kT + threadIdx.x; e < op.n; e += (long long)gridDim.x * kT) {
    double d = 0;
    for (int b = 0; b < B; ++b) {
      const C v = soa ? psi[(long long)b * op.n + e] : psi[e * B + b];
      d += (double)v.x * v.x + (double)v.y * v.y;
    }
    rho[e] = d;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      if (f >= fs.n) break;
      const double b = fs.scale[f] * d;
      const double re = b - apply_op<R>(op, f, fs.x[f], e);
      r[f * op.n + e] = re;
      rr[f] += re * re;
      bb[f] += b * b;
    }
  }
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    if (f >= fs.n) break;
    const double a = block_sum<kT>(rr[f], sh), b = block_sum<kT>(bb[f], sh);
    if (threadIdx.x == 0) {
      part.rr(f)[blockIdx.x] = a;
      part.bb(f)[blockIdx.x] = b;
    }
  }
}

// The start of a field's solve, from the partials of cg_init_kernel: a start
// worse than zero is replaced by zero (r = b, r.r = b.b); convergence test
// r.r <= tol^2 b.b.  Every workgroup decides alike; one stores the scalars.
struct Start {
  bool reset, done;
};
template <int NT>
__device__ __forceinline__ Start solve_start(const Parts& part, int f, int nblk, double tol2, double* __restrict__ scal,
                                             bool store, double* sh) {
  const double rr = sum_partials<NT>(part.rr(f), nblk, sh), bb = sum_partials<NT>(part.bb(f), nblk, sh);
  Start s;
  s.reset = rr > bb;
  s.done = (s.reset ? bb : rr) <= tol2 * bb;
  if (store && threadIdx.x == 0) {
    scal[f * kScal + kBB] = bb;
    scal[f * kScal + kDone] = s.done ? 1.0 : 0.0;
    scal[f * kScal + kIter] = 0.0;
  }
  return s;
}

// ---------------------------------------------------------------------------
// sine transforms on the matrix cores.  S is the symmetric DST-I matrix of an
// axis, zero-padded to n16 x n16 (n16 = n rounded up to 16), so products need
// no bounds.  v_mfma_f64_16x16x4f64: lane l holds A[l & 15][l >> 4],
// B[l >> 4][l & 15] and D[(l >> 4) + 4 v][l & 15].
// ---------------------------------------------------------------------------
typedef double d4 __attribute__((ext_vector_type(4)));

struct Dst {
  const double *sx, *sy, *sz;  // padded matrices
  const double *ex, *ey, *ez;  // eigenvalues
  double norm;
};
__host__ __device__ constexpr int up16(int n) { return (n + 15) & ~15; }
constexpr int kPlaneTiles = 4;  // 16 x 16 tiles per wave at most
constexpr int kPad = 2;         // LDS row padding (doubles)

// acc += S X (LEFT) or X S over k < n16 (a multiple of 16): S from memory (it
// stays in L2) at s, n16 per k, X from LDS at x, sx per k.  The next 16 k of S
// are loaded while the matrix cores work on these.
template <bool LEFT>
__device__ __forceinline__ void mfma_product(const double* s, int n16, const double* x, int sx, d4& acc) {
  double m[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) m[j] = s[4 * j * n16];
  for (int k = 0; k < n16; k += 16) {
    double next[4];
    const int kn = k + 16 < n16 ? k + 16 : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) next[j] = s[(kn + 4 * j) * n16];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double v = x[(k + 4 * j) * sx];
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(LEFT ? m[j] : v, LEFT ? v : m[j], acc, 0, 0, 0);
      m[j] = next[j];
    }
  }
}

// y transform of (x transform of P), P a plane of ny16 rows of nx16 (+ kPad)
// in LDS; tile j of this wave ends in acc[j]
__device__ __forceinline__ void plane_dst(double* P, int nx16, int ny16, const Dst& d, d4* acc) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
  const int ld = nx16 + kPad, ntx = nx16 / 16, nt = ntx * (ny16 / 16);
#pragma unroll
  for (int j = 0; j < kPlaneTiles; ++j) {
    acc[j] = d4{0, 0, 0, 0};
    const int t = w + j * (kPT / 64);
    if (t >= nt) continue;
    mfma_product<false>(d.sx + lk * nx16 + (t % ntx) * 16 + lr, nx16, P + ((t / ntx) * 16 + lr) * ld + lk, 1, acc[j]);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPlaneTiles; ++j) {
    const int t = w + j * (kPT / 64);
    if (t >= nt) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) P[((t / ntx) * 16 + lk + 4 * v) * ld + (t % ntx) * 16 + lr] = acc[j][v];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPlaneTiles; ++j) {
    acc[j] = d4{0, 0, 0, 0};
    const int t = w + j * (kPT / 64);
    if (t >= nt) continue;
    mfma_product<true>(d.sy + lk * ny16 + (t / ntx) * 16 + lr, ny16, P + lk * ld + (t % ntx) * 16 + lr, ld, acc[j]);
  }
}

// plane of `in` (ny rows of nx) into P, zero beyond
__device__ __forceinline__ void plane_load(double* P, const double* __restrict__ in, int nx, int ny, int nx16, int ny16) {
  const int ld = nx16 + kPad, lane = threadIdx.x & 63;
  for (int y = threadIdx.x >> 6; y < ny16; y += kPT / 64)
    for (int x = lane; x < nx16; x += 64) P[y * ld + x] = (y < ny && x < nx) ? in[y * nx + x] : 0.0;
}

// f(index in the plane, value) for this wave's transformed points
template <typename F>
__device__ __forceinline__ void plane_points(const d4* acc, int nx, int ny, int nx16, int ny16, F f) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int ntx = nx16 / 16, nt = ntx * (ny16 / 16);
#pragma unroll
  for (int j = 0; j < kPlaneTiles; ++j) {
    const int t = w + j * (kPT / 64);
    if (t >= nt) continue;
    const int x = (t % ntx) * 16 + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int y = (t / ntx) * 16 + (lane >> 4) + 4 * v;
      if (y < ny && x < nx) f(y * nx + x, acc[j][v]);
    }
  }
}

// x and y transforms of r, plane by plane; with START also the start of the
// solve (x and r replaced where it resets)
template <int CAP, bool START>
__global__ void __launch_bounds__(kPT) dst_planes_kernel(Op op, Fields fs, Dst d, const double* __restrict__ rho,
                                                         double* __restrict__ r, double* __restrict__ t, Parts part,
                                                         int nblk, double tol2, double* __restrict__ scal) {
  __shared__ double P[CAP];
  __shared__ double sh[kPT / 64];
  const int f = blockIdx.y, nx = op.nx, ny = op.ny, nx16 = up16(nx), ny16 = up16(ny);
  const long long plane = (long long)nx * ny, at = f * op.n + blockIdx.x * plane;
  if (START) {
    const Start s = solve_start<kPT>(part, f, nblk, tol2, scal, blockIdx.x == 0, sh);
    if (s.reset) {
      double* x = fs.x[f] + blockIdx.x * plane;
      const double* rh = rho + blockIdx.x * plane;
      for (int i = threadIdx.x; i < plane; i += kPT) {
        x[i] = 0.0;
        r[at + i] = fs.scale[f] * rh[i];
      }
      __syncthreads();
    }
    if (s.done) return;
  } else if (scal[f * kScal + kDone] != 0.0) {
    return;
  }
  plane_load(P, r + at, nx, ny, nx16, ny16);
  __syncthreads();
  d4 acc[kPlaneTiles];
  plane_dst(P, nx16, ny16, d, acc);
  plane_points(acc, nx, ny, nx16, ny16, [&](int i, double v) { t[at + i] = v; });
}

// the same back: t to the preconditioned residual z, and the plane's part of
// r.z
template <int CAP>
__global__ void __launch_bounds__(kPT) dst_planes_back_kernel(Op op, Dst d, const double* __restrict__ t,
                                                              const double* __restrict__ r, double* __restrict__ z,
                                                              Parts part, const double* __restrict__ scal) {
  __shared__ double P[CAP];
  __shared__ double sh[kPT / 64];
  const int f = blockIdx.y, nx = op.nx, ny = op.ny, nx16 = up16(nx), ny16 = up16(ny);
  const long long at = f * op.n + (long long)blockIdx.x * nx * ny;
  if (scal[f * kScal + kDone] != 0.0) return;
  plane_load(P, t + at, nx, ny, nx16, ny16);
  __syncthreads();
  d4 acc[kPlaneTiles];
  plane_dst(P, nx16, ny16, d, acc);
  double rz = 0;
  plane_points(acc, nx, ny, nx16, ny16, [&](int i, double v) {
    z[at + i] = v;
    rz += r[at + i] * v;
  });
  rz = block_sum<kPT>(rz, sh);
  if (threadIdx.x == 0) part.rz(f)[blockIdx.x] = rz;
}

// z transform, division by the eigenvalues of the R = 1 operator (times the
// transforms' normalisation) and z transform back, in place: 16 columns of
// the (y, x) plane per workgroup, its waves taking 16-row tiles in turn
constexpr int kZT = 256, kZRows = 256, kZTiles = kZRows / 16 / (kZT / 64);
__global__ void __launch_bounds__(kZT) dst_columns_kernel(Op op, Fields fs, Dst d, double* __restrict__ t,
                                                          const double* __restrict__ scal) {
  constexpr int LD = 16 + kPad;
  __shared__ double X[kZRows * LD];
  const int f = blockIdx.y, nz = op.nz, nz16 = up16(nz);
  if (scal[f * kScal + kDone] != 0.0) return;
  const long long ncol = (long long)op.nx * op.ny, c0 = 16LL * blockIdx.x;
  double* tf = t + f * op.n;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
  const double* s0 = d.sz + lk * nz16 + lr;
  for (int i = threadIdx.x; i < nz16 * 16; i += kZT) {
    const int k = i >> 4, c = i & 15;
    X[k * LD + c] = (k < nz && c0 + c < ncol) ? tf[k * ncol + c0 + c] : 0.0;
  }
  const long long col = c0 + lr;
  const bool in = col < ncol;
  const int iy = in ? (int)(col / op.nx) : 0, ix = in ? (int)(col - (long long)iy * op.nx) : 0;
  const double exy = d.ex[ix] + d.ey[iy] + fs.mu2[f];
  __syncthreads();
  d4 acc[kZTiles];
  for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
    for (int j = 0; j < kZTiles; ++j) {
      acc[j] = d4{0, 0, 0, 0};
      const int m = 16 * (w + j * (kZT / 64));
      if (m >= nz16) continue;
      mfma_product<true>(s0 + m, nz16, X + lk * LD + lr, LD, acc[j]);
    }
    if (pass == 1) break;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kZTiles; ++j) {
      const int m = 16 * (w + j * (kZT / 64));
      if (m >= nz16) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = m + lk + 4 * v;
        X[k * LD + lr] = k < nz ? acc[j][v] * (d.norm / (exy + d.ez[k])) : 0.0;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < kZTiles; ++j) {
    const int m = 16 * (w + j * (kZT / 64));
    if (m >= nz16) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = m + lk + 4 * v;
      if (k < nz && in) tf[k * ncol + col] = acc[j][v];
    }
  }
}

// ---------------------------------------------------------------------------
// planes beyond LDS: rocBLAS GEMMs
// ---------------------------------------------------------------------------

// the start of the solve on its own (one workgroup per block of points)
__global__ void __launch_bounds__(kT) cg_start_kernel(Op op, Fields fs, const double* __restrict__ rho,
                                                      double* __restrict__ r, Parts part, int nblk, double tol2,
                                                      double* __restrict__ scal) {
  __shared__ double sh[kT / 64];
  const int f = blockIdx.y;
  const Start s = solve_start<kT>(part, f, nblk, tol2, scal, blockIdx.x == 0, sh);
  if (!s.reset) return;
  for (long long e = (long long)blockIdx.x * kT + threadIdx.x; e < op.n; e += (long long)gridDim.x * kT) {
    fs.x[f][e] = 0.0;
    r[f * op.n + e] = fs.scale[f] * rho[e];
  }
}

// partials of r.z
__global__ void __launch_bounds__(kT) cg_dot_kernel(Op op, const double* __restrict__ r, const double* __restrict__ z,
                                                    Parts part, const double* __restrict__ scal) {
  __shared__ double sh[kT / 64];
  const int f = blockIdx.y;
  if (scal[f * kScal + kDone] != 0.0) return;
  double rz = 0;
  for (long long e = (long long)blockIdx.x * kT + threadIdx.x; e < op.n; e += (long long)gridDim.x * kT)
    rz += r[f * op.n + e] * z[f * op.n + e];
  rz = block_sum<kT>(rz, sh);
  if (threadIdx.x == 0) part.rz(f)[blockIdx.x] = rz;
}

// divide the sine coefficients by the eigenvalues of the R = 1 operator
// (-Delta_h + mu^2, zero outside) times the transforms' normalisation
__global__ void __launch_bounds__(kT) dst_scale_kernel(Op op, Dst d, double mu2, double* __restrict__ a) {
  const long long e = (long long)blockIdx.x * kT + threadIdx.x;
  if (e >= op.n) return;
  const int ix = (int)(e % op.nx), iy = (int)((e / op.nx) % op.ny), iz = (int)(e / ((long long)op.nx * op.ny));
  a[e] *= d.norm / (d.ex[ix] + d.ey[iy] + d.ez[iz] + mu2);
}

// One sine transform of [z][y][x] data along all three axes: three FP64
// GEMMs with the symmetric DST-I matrices (x: S_x X; y: per z-plane X S_y;
// z: X S_z in the column-major views), in -> out through tmp.
rocblas_status dst3(const PotentialSolver& ps, const double* in, double* tmp, double* out) {
  rocblas_handle hb = static_cast<rocblas_handle>(ps.blas);
  const int nx = ps.nx, ny = ps.ny, nz = ps.nz;
  const double one = 1.0, zero = 0.0;
  rocblas_status rs = rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, nx, ny * nz, nx, &one, ps.sx,
                                    up16(nx), in, nx, &zero, out, nx);
  if (rs == rocblas_status_success)
    rs = rocblas_dgemm_strided_batched(hb, rocblas_operation_none, rocblas_operation_none, nx, ny, ny, &one, out, nx,
                                       (rocblas_stride)nx * ny, ps.sy, up16(ny), 0, &zero, tmp, nx,
                                       (rocblas_stride)nx * ny, nz);
  if (rs == rocblas_status_success)
    rs = rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, nx * ny, nz, nz, &one, tmp, nx * ny, ps.sz,
                       up16(nz), &zero, out, nx * ny);
  return rs;
}

// ---------------------------------------------------------------------------
// the iteration
// ---------------------------------------------------------------------------

// q = A p; partials of p.q
template <int R>
__global__ void __launch_bounds__(kT) cg_ap_kernel(Op op, const double* __restrict__ p, double* __restrict__ q,
                                                   Parts part, const double* __restrict__ scal) {
  __shared__ double sh[kT / 64];
  const int f = blockIdx.y;
  if (scal[f * kScal + kDone] != 0.0) return;
  p += f * op.n;
  q += f * op.n;
  double pq = 0;
  for (long long e = (long long)blockIdx.x * kT + threadIdx.x; e < op.n; e += (long long)gridDim.x * kT) {
    const double v = apply_op<R>(op, f, p, e);
    q[e] = v;
    pq += p[e] * v;
  }
  pq = block_sum<kT>(pq, sh);
  if (threadIdx.x == 0) part.pq(f)[blockIdx.x] = pq;
}

// alpha = (r.z) / (p.q); x += alpha p; r -= alpha q; partials of r.r.
// `nrz` partials of r.z, kept as the scalar r.z for the next direction.
__global__ void __launch_bounds__(kT) cg_x_kernel(Op op, Fields fs, double* __restrict__ r,
                                                  const double* __restrict__ p, const double* __restrict__ q,
                                                  Parts part, int nrz, double* __restrict__ scal) {
  __shared__ double sh[kT / 64];
  const int f = blockIdx.y;
  if (scal[f * kScal + kDone] != 0.0) return;
  const double pq = sum_partials<kT>(part.pq(f), gridDim.x, sh), rz = sum_partials<kT>(part.rz(f), nrz, sh);
  if (blockIdx.x == 0 && threadIdx.x == 0) scal[f * kScal + kRZ] = rz;
  const double alpha = rz / pq;
  double* x = fs.x[f];
  r += f * op.n;
  p += f * op.n;
  q += f * op.n;
  double rr = 0;
  for (long long e = (long long)blockIdx.x * kT + threadIdx.x; e < op.n; e += (long long)gridDim.x * kT) {
    x[e] += alpha * p[e];
    const double re = r[e] - alpha * q[e];
    r[e] = re;
    rr += re * re;
  }
  rr = block_sum<kT>(rr, sh);
  if (threadIdx.x == 0) part.rr(f)[blockIdx.x] = rr;
}

// end of an iteration (one workgroup per field): the count and convergence
// on r.r; `host` (pinned, or null) receives the flag and the count
__global__ void __launch_bounds__(kT) cg_check_kernel(Parts part, int nblk, double tol2, double* __restrict__ scal,
                                                      double* __restrict__ host) {
  __shared__ double sh[kT / 64];
  const int f = blockIdx.x;
  double* sc = scal + f * kScal;
  bool done = sc[kDone] != 0.0;
  double it = sc[kIter];
  const double rr = sum_partials<kT>(part.rr(f), nblk, sh);
  if (threadIdx.x != 0) return;
  if (!done) {
    done = rr <= tol2 * sc[kBB];
    it += 1.0;
    sc[kIter] = it;
    sc[kDone] = done ? 1.0 : 0.0;
  }
  if (host) {
    host[2 * f + 1] = it;
    __hip_atomic_store(&host[2 * f], done ? 1.0 : 0.0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// beta = (r'.z') / (r.z); p = z + beta p
__global__ void __launch_bounds__(kT) cg_p_kernel(Op op, double* __restrict__ p, const double* __restrict__ z,
                                                  Parts part, int nrz, const double* __restrict__ scal) {
  __shared__ double sh[kT / 64];
  const int f = blockIdx.y;
  if (scal[f * kScal + kDone] != 0.0) return;
  const double beta = sum_partials<kT>(part.rz(f), nrz, sh) / scal[f * kScal + kRZ];
  p += f * op.n;
  z += f * op.n;
  for (long long e = (long long)blockIdx.x * kT + threadIdx.x; e < op.n; e += (long long)gridDim.x * kT)
    p[e] = z[e] + beta * p[e];
}

Dst make_dst(const PotentialSolver& ps) {
  Dst d{};
  d.sx = ps.sx;
  d.sy = ps.sy;
  d.sz = ps.sz;
  d.ex = ps.ex;
  d.ey = ps.ey;
  d.ez = ps.ez;
  d.norm = (2.0 / (ps.nx + 1)) * (2.0 / (ps.ny + 1)) * (2.0 / (ps.nz + 1));
  return d;
}

// LDS doubles of a plane, by class (33, 75 and 130 KiB); 0: beyond
constexpr int kCap[3] = {64 * (64 + kPad), 96 * (96 + kPad), 128 * (128 + kPad)};
int plane_cap(const PotentialSolver& ps) {
  const int nx16 = up16(ps.nx), ny16 = up16(ps.ny);
  if ((nx16 / 16) * (ny16 / 16) > kPlaneTiles * (kPT / 64) || up16(ps.nz) > kZRows) return 0;
  for (int cap : kCap)
    if (ny16 * (nx16 + kPad) <= cap) return cap;
  return 0;
}

// z = M^{-1} r with M the R = 1 operator (exact for R = 1, spectrally
// equivalent for R = 2, 3) and the partials of r.z; with `start` the solve's
// start before it
template <int CAP>
void precond_planes(const PotentialSolver& ps, const Op& op, const Fields& fs, const Parts& part, bool start, double* z,
                    hipStream_t st) {
  const Dst d = make_dst(ps);
  const dim3 gp(ps.nz, fs.n), gc((unsigned)(((long long)ps.nx * ps.ny + 15) / 16), fs.n);
  const double tol2 = ps.tol * ps.tol;
  if (start)
    dst_planes_kernel<CAP, true><<<gp, kPT, 0, st>>>(op, fs, d, ps.rho, ps.r, ps.t1, part, ps.nblk, tol2, ps.scal);
  else
    dst_planes_kernel<CAP, false><<<gp, kPT, 0, st>>>(op, fs, d, ps.rho, ps.r, ps.t1, part, ps.nblk, tol2, ps.scal);
  dst_columns_kernel<<<gc, kZT, 0, st>>>(op, fs, d, ps.t1, ps.scal);
  dst_planes_back_kernel<CAP><<<gp, kPT, 0, st>>>(op, d, ps.t1, ps.r, z, part, ps.scal);
}

hipError_t precond(const PotentialSolver& ps, const Op& op, const Fields& fs, const Parts& part, bool start, double* z,
                   hipStream_t st) {
  switch (plane_cap(ps)) {
    case kCap[0]: precond_planes<kCap[0]>(ps, op, fs, part, start, z, st); return hipGetLastError();
    case kCap[1]: precond_planes<kCap[1]>(ps, op, fs, part, start, z, st); return hipGetLastError();
    case kCap[2]: precond_planes<kCap[2]>(ps, op, fs, part, start, z, st); return hipGetLastError();
    default: break;
  }
  const Dst d = make_dst(ps);
  const dim3 g(ps.nblk, fs.n);
  if (start)
    cg_start_kernel<<<g, kT, 0, st>>>(op, fs, ps.rho, ps.r, part, ps.nblk, ps.tol * ps.tol, ps.scal);
  if (rocblas_set_stream(static_cast<rocblas_handle>(ps.blas), st) != rocblas_status_success) return hipErrorUnknown;
  for (int f = 0; f < fs.n; ++f) {
    if (dst3(ps, ps.r + f * op.n, ps.t1, ps.t2) != rocblas_status_success) return hipErrorLaunchFailure;
    dst_scale_kernel<<<(unsigned)((op.n + kT - 1) / kT), kT, 0, st>>>(op, d, fs.mu2[f], ps.t2);
    if (dst3(ps, ps.t2, ps.t1, z + f * op.n) != rocblas_status_success) return hipErrorLaunchFailure;
  }
  cg_dot_kernel<<<g, kT, 0, st>>>(op, ps.r, z, part, ps.scal);
  return hipGetLastError();
}

Op make_op(const PotentialSolver& ps, const Fields& fs) {
  Op op{};
  op.nx = ps.nx;
  op.ny = ps.ny;
  op.nz = ps.nz;
  op.n = (long long)ps.nx * ps.ny * ps.nz;
  const double ih2 = 1.0 / (ps.h * ps.h);
  for (int f = 0; f < fs.n; ++f) op.diag[f] = -3.0 * ps.c[0] * ih2 + fs.mu2[f];
  for (int k = 1; k <= ps.R; ++k) op.off[k] = -ps.c[k] * ih2;
  return op;
}

// the fields that are switched on: Yukawa, then Coulomb
Fields make_fields(const PotentialSolver& ps) {
  Fields fs{};
  if (ps.v0 != 0.0) {
    fs.mu2[fs.n] = 1.0 / (ps.a * ps.a);
    fs.scale[fs.n] = 4.0 * M_PI * ps.v0 * ps.a;
    fs.x[fs.n++] = ps.wy;
  }
  if (ps.e2 != 0.0) {
    fs.mu2[fs.n] = 0.0;
    fs.scale[fs.n] = 2.0 * M_PI * ps.e2;
    fs.x[fs.n++] = ps.wc;
  }
  return fs;
}

// Waits until the flags of this iteration have arrived in pinned memory: all
// work queued before them is done then.  The host polls them, a few
// microseconds sooner than the stream's own synchronisation returns, for at
// most 5 ms; after that (a long queue before this solve, or an error) it
// synchronises the stream.  Either takes the core meanwhile (a step behind 28 ms
// of queued work: 28.4 ms of CPU time, 28.8 with the synchronisation alone).
hipError_t wait_flags(const PotentialSolver& ps, int nf, hipStream_t st) {
  const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(5);
  auto arrived = [&]() {
    for (int f = 0; f < nf; ++f)
      if (__atomic_load_n(reinterpret_cast<long long*>(&ps.host[2 * f]), __ATOMIC_ACQUIRE) == kPending) return false;
    return true;
  };
  while (!arrived()) {
    if (std::chrono::steady_clock::now() < until) continue;
    return hipStreamSynchronize(st);
  }
  return hipSuccess;
}

// density and both solves
template <typename C, int R>
hipError_t solve_fields(PotentialSolver& ps, const void* psi, bool soa, int B, hipStream_t st) {
  const Fields fs = make_fields(ps);
  const Op op = make_op(ps, fs);
  const Parts part{ps.part, std::max(ps.nblk, ps.nz)};
  const int nrz = plane_cap(ps) ? ps.nz : ps.nblk;
  const double tol2 = ps.tol * ps.tol;
  const dim3 g(ps.nblk, std::max(fs.n, 1));
  cg_init_kernel<C, R><<<ps.nblk, kT, 0, st>>>(op, static_cast<const C*>(psi), B, soa ? 1 : 0, ps.rho, fs, ps.r, part);
  hipError_t e = hipGetLastError();
  if (fs.n == 0) {
    if (e == hipSuccess) ++ps.solves;
    return e;
  }
  // the first direction is the preconditioned residual itself
  if (e == hipSuccess) e = precond(ps, op, fs, part, true, ps.p, st);
  const int most = ps.fixed > 0 ? ps.fixed : ps.maxit;
  for (int it = 0; e == hipSuccess && it < most; ++it) {
    if (it > 0) {
      e = precond(ps, op, fs, part, false, ps.z, st);
      if (e != hipSuccess) break;
      cg_p_kernel<<<g, kT, 0, st>>>(op, ps.p, ps.z, part, nrz, ps.scal);
    }
    cg_ap_kernel<R><<<g, kT, 0, st>>>(op, ps.p, ps.q, part, ps.scal);
    cg_x_kernel<<<g, kT, 0, st>>>(op, fs, ps.r, ps.p, ps.q, part, nrz, ps.scal);
    for (int f = 0; f < fs.n && ps.fixed == 0; ++f)
      __atomic_store_n(reinterpret_cast<long long*>(&ps.host[2 * f]), kPending, __ATOMIC_RELAXED);
    cg_check_kernel<<<fs.n, kT, 0, st>>>(part, ps.nblk, tol2, ps.scal, ps.fixed > 0 ? nullptr : ps.host);
    e = hipGetLastError();
    if (ps.fixed > 0) continue;
    // few iterations with this preconditioner: read the flags after each
    if (e == hipSuccess) e = wait_flags(ps, fs.n, st);
    if (e == hipSuccess && ps.host[0] != 0.0 && (fs.n == 1 || ps.host[2] != 0.0)) break;
  }
  if (e == hipSuccess && ps.fixed == 0) {
    int f = 0;
    if (ps.v0 != 0.0) ps.iters_y += (long long)ps.host[2 * f++ + 1];
    if (ps.e2 != 0.0) ps.iters_c += (long long)ps.host[2 * f + 1];
  }
  if (e == hipSuccess) ++ps.solves;
  return e;
}

// the potential, and at the end of the solves their iterations into
// tally[0] (Yukawa) and tally[1] (Coulomb), unconverged ones into tally[2]
template <typename T>
__global__ void __launch_bounds__(kT) veff_kernel(const T* __restrict__ V, const double* __restrict__ rho,
                                                  const double* __restrict__ wy, const double* __restrict__ wc,
                                                  long long n, double t0, double t3, T* __restrict__ veff,
                                                  const double* __restrict__ scal, double* __restrict__ tally) {
  const long long p = (long long)blockIdx.x * kT + threadIdx.x;
  if (p == 0) {
    int f = 0;
    for (int k = 0; k < 2; ++k) {
      if (!(k == 0 ? wy : wc)) continue;
      tally[k] += scal[f * kScal + kIter];
      if (scal[f * kScal + kDone] == 0.0) tally[2] += 1.0;
      ++f;
    }
  }
  if (p >= n) return;
  const double r = rho[p];
  double u = t0 * r + t3 * r * r;
  if (wy) u += wy[p];
  if (wc) u += wc[p];
  veff[p] = (T)((V ? (double)V[p] : 0.0) + u);
}

template <typename C>
hipError_t solve_radius(PotentialSolver& ps, const void* psi, bool soa, int B, hipStream_t st) {
  switch (ps.R) {
    case 1: return solve_fields<C, 1>(ps, psi, soa, B, st);
    case 2: return solve_fields<C, 2>(ps, psi, soa, B, st);
    case 3: return solve_fields<C, 3>(ps, psi, soa, B, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool potential_needs_blas(const PotentialSolver& ps) { return plane_cap(ps) == 0; }

// one transform pair on zero data at setup, so that rocBLAS (where the
// transforms need it) finishes its lazy initialisation before the first step
hipError_t potential_warmup(PotentialSolver& ps) {
  if (!potential_needs_blas(ps)) return hipSuccess;
  const size_t n = (size_t)ps.nx * ps.ny * ps.nz;
  hipError_t e = hipMemset(ps.r, 0, n * sizeof(double));
  if (e != hipSuccess) return e;
  if (rocblas_set_stream(static_cast<rocblas_handle>(ps.blas), nullptr) != rocblas_status_success)
    return hipErrorUnknown;
  if (dst3(ps, ps.r, ps.t1, ps.t2) != rocblas_status_success) return hipErrorLaunchFailure;
  return hipDeviceSynchronize();
}

// V + t0 rho + t3 rho^2 + W_Y + W_C for the state psi (AoS [point][orbital]
// or SoA [orbital][point] orbital arrays), into veff of the state's real type
hipError_t skyrme_veff(PotentialSolver& ps, const void* psi, bool soa, int B, bool c64, const void* V, void* veff,
                       double t0, double t3, hipStream_t st, abc_timer* tm) {
  const long long n = (long long)ps.nx * ps.ny * ps.nz;
  const unsigned blocks = (unsigned)((n + kT - 1) / kT);
  const hipError_t e = c64 ? solve_radius<float2>(ps, psi, soa, B, st) : solve_radius<double2>(ps, psi, soa, B, st);
  if (e != hipSuccess) return e;
  const double* wy = ps.v0 != 0.0 ? ps.wy : nullptr;
  const double* wc = ps.e2 != 0.0 ? ps.wc : nullptr;
  if (c64)
    abc_launch_kernel(tm, "meanfield", veff_kernel<float>, dim3(blocks), dim3(kT), st, static_cast<const float*>(V),
                      (const double*)ps.rho, wy, wc, n, t0, t3, static_cast<float*>(veff), (const double*)ps.scal,
                      ps.tally);
  else
    abc_launch_kernel(tm, "meanfield", veff_kernel<double>, dim3(blocks), dim3(kT), st,
                      static_cast<const double*>(V), (const double*)ps.rho, wy, wc, n, t0, t3,
                      static_cast<double*>(veff), (const double*)ps.scal, ps.tally);
  return hipGetLastError();
}
