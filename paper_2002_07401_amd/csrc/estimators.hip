// Force and optimisation estimators on top of the adjoint's per-walker
// derivatives (Atomic forces and Stochastic reconfiguration sections).
//
// * Space warp: omega_a(r) = kappa_a / sum_b kappa_b, kappa = 1/|r - R|^4;
//   total derivatives dR_a + sum_i omega_a(r_i) dr_i (+ 1/2 sum_i grad omega_a(r_i)
//   for ln(J^1/2 Psi)), one workgroup per walker.
// * Finite-variance reweighting: R = (S sum_ij (W^-1)_ij^2)^(-theta),
//   S = min_i sum_j W_ij^2, weight = (R / max(R, eps))^2, one workgroup per walker
//   (W the geminal matrix, or the Pfaffian's pairing matrix G~).
// * Stochastic reconfiguration: (S + eps diag S) delta = f with
//   S v = O^T (w o (O v)) / sum w - Obar (Obar . v), f = -2 sum_i w_i e_i (O_i - Obar) / sum w,
//   solved by diagonally preconditioned conjugate gradients on the device
//   without forming S: per iteration u = O p (and Obar . p), O^T (w o u) by
//   column slices, S' p with partial sums of p . S'p, the x / r update with
//   partial sums of r . z and r . r, the p update.  Every reduction is a fixed-order sum
//   of per-block partials; the iteration scalars are double-buffered by parity
//   so no block reads a value another block of the same launch writes.
#include <mutex>

#include "internal.h"

namespace qmc {

// ---------------------------------------------------------------------------
// space warp
// ---------------------------------------------------------------------------
constexpr int kSwctMaxN = 1024;

__global__ void __launch_bounds__(256)
swct_kernel(SysDev s, const double* __restrict__ r, const double* __restrict__ dR, const double* __restrict__ dr,
            int jac, double* __restrict__ out) {
  __shared__ double K[kSwctMaxN][4];   // sum_b kappa_b and its gradient, per electron
  const int wk = blockIdx.x, N = s.N, A = s.n_nuc;
  const double* rw = r + (long)wk * N * 3;
  for (int i = threadIdx.x; i < N; i += blockDim.x) {
    double k0 = 0.0, kx = 0.0, ky = 0.0, kz = 0.0;
    for (int b = 0; b < A; ++b) {
      const double dx = rw[3 * i] - s.R[3 * b], dy = rw[3 * i + 1] - s.R[3 * b + 1], dz = rw[3 * i + 2] - s.R[3 * b + 2];
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double ik = 1.0 / (r2 * r2);
      const double g = -4.0 * ik / r2;
      k0 += ik; kx += g * dx; ky += g * dy; kz += g * dz;
    }
    K[i][0] = k0; K[i][1] = kx; K[i][2] = ky; K[i][3] = kz;
  }
  __syncthreads();
  const double* drw = dr + (long)wk * N * 3;
  for (int a = threadIdx.x; a < A; a += blockDim.x) {
    double t0 = 0.0, t1 = 0.0, t2 = 0.0, j0 = 0.0, j1 = 0.0, j2 = 0.0;
    for (int i = 0; i < N; ++i) {
      const double dx = rw[3 * i] - s.R[3 * a], dy = rw[3 * i + 1] - s.R[3 * a + 1], dz = rw[3 * i + 2] - s.R[3 * a + 2];
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double ka = 1.0 / (r2 * r2);
      const double om = ka / K[i][0];
      t0 += om * drw[3 * i]; t1 += om * drw[3 * i + 1]; t2 += om * drw[3 * i + 2];
      if (jac) {
        const double g = -4.0 * ka / r2, iK = 1.0 / K[i][0];
        j0 += g * dx * iK - ka * K[i][1] * iK * iK;
        j1 += g * dy * iK - ka * K[i][2] * iK * iK;
        j2 += g * dz * iK - ka * K[i][3] * iK * iK;
      }
    }
    const double* dRa = dR + ((long)wk * A + a) * 3;
    double* o = out + ((long)wk * A + a) * 3;
    o[0] = dRa[0] + t0 + 0.5 * j0;
    o[1] = dRa[1] + t1 + 0.5 * j1;
    o[2] = dRa[2] + t2 + 0.5 * j2;
  }
}

hipError_t launch_swct(const SysDev& s, int Wk, const double* r, const double* dR, const double* dr, int jac,
                       double* out, hipStream_t st) {
  if (s.N > kSwctMaxN) return hipErrorNotSupported;
  hipLaunchKernelGGL(swct_kernel, dim3(Wk), dim3(256), 0, st, s, r, dR, dr, jac, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// reweighting factor
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
reweight_kernel(SysDev s, WalkDev w, double theta, double eps, double* __restrict__ Rout,
                double* __restrict__ wout) {
  __shared__ double red[4], redm[4];
  // the pairing matrix: W (n_up x n_up), or G~ of the Pfaffian with its exact inverse
  const int wk = blockIdx.x, n = s.pairing ? s.npf : s.nu, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double* W = w.W + (long)wk * n * n;
  const double* A = w.A + (long)wk * n * n;
  double smin = __builtin_inf(), sa = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double rs = 0.0;
    for (int j = 0; j < n; ++j) rs += W[(long)i * n + j] * W[(long)i * n + j];
    smin = fmin(smin, rs);
  }
  for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) sa += A[idx] * A[idx];
  sa = wave_sum(sa);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) smin = fmin(smin, __shfl_xor(smin, o, 64));
  if (lane == 0) { red[wave] = sa; redm[wave] = smin; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0, m = __builtin_inf();
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) { t += red[k]; m = fmin(m, redm[k]); }
    const double R = pow(m * t, -theta);
    const double Re = fmax(R, eps);
    Rout[wk] = R;
    if (wout) wout[wk] = (R / Re) * (R / Re);
  }
}

hipError_t launch_reweight(const SysDev& s, const WalkDev& w, double theta, double eps, double* R, double* weight,
                           hipStream_t st) {
  hipLaunchKernelGGL(reweight_kernel, dim3(w.Wk), dim3(256), 0, st, s, w, theta, eps, R, weight);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// stochastic reconfiguration
// ---------------------------------------------------------------------------
// Conjugate gradients preconditioned by the diagonal of S' (m_k = (1 + eps) s_kk,
// 1 where s_kk = 0): the regularisation is relative to the diagonal, so the
// diagonally scaled matrix has unit diagonal and a condition number bounded by
// about (P + eps) / eps whatever the scales of the parameters.
// The column sums over samples (moments, O^T (w o u)) run on a 2-D grid:
// blocks of 256 columns times `ms` slices of the samples, each slice writing
// its partial sums, which a second kernel adds in slice order.
// Workspace of the two-pass path (doubles): Obar, d (= diag S), f, r, p, Sp [P each], u [M],
// part1, part2, part3 [nblk each], colpart [2][ms][P], scalars [16]:
//   sc[0] = sum w, sc[1] = f . f, sc[2 + (it & 1)] = r . z at iteration it,
//   sc[4] = Obar . p, sc[5] = done, sc[6] = r . r of the last update
struct SrWork {
  double *Obar, *d, *f, *r, *p, *Sp, *u, *part1, *part2, *part3, *colpart, *sc;
  long P;
  int M, nblk, ms, rows;   // rows: samples per slice
  double eps;
};

static int sr_slices(int M) {
  const int ms = (M + 127) / 128;   // about 128 samples per slice, at most 64 slices
  return ms < 1 ? 1 : (ms > 64 ? 64 : ms);
}

__device__ inline double sr_precond(const SrWork& q, long k) {
  const double m = (1.0 + q.eps) * q.d[k];
  return m > 0.0 ? m : 1.0;
}

__device__ double blk_sum256(double v, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int k = 0; k < 4; ++k) t += red[k];
  __syncthreads();
  return t;
}

// sum of the weights (single workgroup)
__global__ void __launch_bounds__(256) sr_wsum_kernel(SrWork q, const double* __restrict__ wts) {
  __shared__ double red[4];
  double t = 0.0;
  for (int i = threadIdx.x; i < q.M; i += blockDim.x) t += wts ? wts[i] : 1.0;
  t = blk_sum256(t, red);
  if (threadIdx.x == 0) q.sc[0] = t;
}

// (The loops below are unrolled for their loads alone: the sums keep their order.)
// Column sums over one slice of samples: pass 0: sum w O; pass 1: sum w (O - Obar)^2
// and sum w e (O - Obar); pass 2: sum w u O (u = O p).
__global__ void __launch_bounds__(256)
sr_colsum_kernel(SrWork q, const double* __restrict__ O, const double* __restrict__ el,
                 const double* __restrict__ wts, int pass) {
  if (pass == 2 && q.sc[5] != 0.0) return;   // converged (uniform)
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int sl = blockIdx.y;
  if (k >= q.P) return;
  const int i0 = sl * q.rows, i1 = min(i0 + q.rows, q.M);
  double a = 0.0, b = 0.0;
  if (pass == 0) {
#pragma unroll 16
    for (int i = i0; i < i1; ++i) a += (wts ? wts[i] : 1.0) * O[(long)i * q.P + k];
  } else if (pass == 1) {
    const double m = q.Obar[k];
#pragma unroll 8
    for (int i = i0; i < i1; ++i) {
      const double wi = wts ? wts[i] : 1.0, c = O[(long)i * q.P + k] - m;
      a += wi * c * c;
      b += wi * el[i] * c;
    }
  } else {
#pragma unroll 16
    for (int i = i0; i < i1; ++i) a += (wts ? wts[i] : 1.0) * q.u[i] * O[(long)i * q.P + k];
  }
  q.colpart[(long)sl * q.P + k] = a;
  if (pass == 1) q.colpart[((long)q.ms + sl) * q.P + k] = b;
}

// Obar = (sum over slices) / sum w
__global__ void __launch_bounds__(256) sr_mean_kernel(SrWork q) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= q.P) return;
  double a = 0.0;
  for (int sl = 0; sl < q.ms; ++sl) a += q.colpart[(long)sl * q.P + k];
  q.Obar[k] = a / q.sc[0];
}

// diag S and f; x = 0, r = f, p = z = f / m; partial sums of r . z and r . r
__global__ void __launch_bounds__(256) sr_moments_kernel(SrWork q, double* __restrict__ x) {
  __shared__ double red[4];
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  double rz = 0.0, rr = 0.0;
  if (k < q.P) {
    const double iw = 1.0 / q.sc[0];
    double s2 = 0.0, fe = 0.0;
    for (int sl = 0; sl < q.ms; ++sl) {
      s2 += q.colpart[(long)sl * q.P + k];
      fe += q.colpart[((long)q.ms + sl) * q.P + k];
    }
    const double f = -2.0 * fe * iw;
    q.d[k] = s2 * iw; q.f[k] = f;
    const double z = f / sr_precond(q, k);
    q.r[k] = f; q.p[k] = z; x[k] = 0.0;
    rz = f * z;
    rr = f * f;
  }
  rz = blk_sum256(rz, red);
  rr = blk_sum256(rr, red);
  if (threadIdx.x == 0) { q.part2[blockIdx.x] = rz; q.part3[blockIdx.x] = rr; }
}

// r0 . z0 and f . f (single workgroup, fixed order)
__global__ void __launch_bounds__(64) sr_init_kernel(SrWork q) {
  if (threadIdx.x != 0) return;
  double rz = 0.0, rr = 0.0;
  for (int b = 0; b < q.nblk; ++b) { rz += q.part2[b]; rr += q.part3[b]; }
  q.sc[1] = rr;
  q.sc[2] = rz;
  q.sc[6] = rr;
  q.sc[5] = rr > 0.0 ? 0.0 : 1.0;
}

// u_i = O_i . p (workgroups 0..M-1) and Obar . p (workgroup M)
__global__ void __launch_bounds__(256) sr_op_kernel(SrWork q, const double* __restrict__ O) {
  __shared__ double red[4];
  if (q.sc[5] != 0.0) return;   // converged (uniform)
  const int i = blockIdx.x;
  const double* row = i < q.M ? O + (long)i * q.P : q.Obar;
  double t = 0.0;
#pragma unroll 8
  for (long k = threadIdx.x; k < q.P; k += 256) t += row[k] * q.p[k];
  t = blk_sum256(t, red);
  if (threadIdx.x == 0) {
    if (i < q.M) q.u[i] = t;
    else q.sc[4] = t;
  }
}

// element k of S'p from t = (O^T (w o u))_k
__device__ inline double sr_sp(const SrWork& q, long k, double t, double pk) {
  return t / q.sc[0] - q.Obar[k] * q.sc[4] + q.eps * q.d[k] * pk;
}

// S'p from the slice sums of O^T (w o u), and partial sums of p . S'p
__global__ void __launch_bounds__(256) sr_sp_kernel(SrWork q) {
  __shared__ double red[4];
  if (q.sc[5] != 0.0) return;
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  double pp = 0.0;
  if (k < q.P) {
    double t = 0.0;
    for (int sl = 0; sl < q.ms; ++sl) t += q.colpart[(long)sl * q.P + k];
    const double sp = sr_sp(q, k, t, q.p[k]);
    q.Sp[k] = sp;
    pp = q.p[k] * sp;
  }
  pp = blk_sum256(pp, red);
  if (threadIdx.x == 0) q.part1[blockIdx.x] = pp;
}

// alpha = r.z / p.S'p; x += alpha p; r -= alpha S'p; partial sums of r . z and r . r
__global__ void __launch_bounds__(256) sr_update_kernel(SrWork q, double* __restrict__ x, int it) {
  __shared__ double red[4];
  __shared__ double alpha_s;
  if (q.sc[5] != 0.0) return;
  if (threadIdx.x == 0) {
    double pSp = 0.0;
    for (int b = 0; b < q.nblk; ++b) pSp += q.part1[b];
    alpha_s = pSp > 0.0 ? q.sc[2 + (it & 1)] / pSp : 0.0;
  }
  __syncthreads();
  const double alpha = alpha_s;
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  double rz = 0.0, rr = 0.0;
  if (k < q.P) {
    x[k] += alpha * q.p[k];
    const double rk = q.r[k] - alpha * q.Sp[k];
    q.r[k] = rk;
    rz = rk * rk / sr_precond(q, k);
    rr = rk * rk;
  }
  rz = blk_sum256(rz, red);
  rr = blk_sum256(rr, red);
  if (threadIdx.x == 0) { q.part2[blockIdx.x] = rz; q.part3[blockIdx.x] = rr; }
}

// beta = r.z(new) / r.z(old); p = z + beta p
__global__ void __launch_bounds__(256) sr_dir_kernel(SrWork q, int it) {
  __shared__ double beta_s, rzn_s, rrn_s;
  if (q.sc[5] != 0.0) return;
  if (threadIdx.x == 0) {
    double rzn = 0.0, rrn = 0.0;
    for (int b = 0; b < q.nblk; ++b) { rzn += q.part2[b]; rrn += q.part3[b]; }
    const double rzo = q.sc[2 + (it & 1)];
    beta_s = rzo > 0.0 ? rzn / rzo : 0.0;
    rzn_s = rzn;
    rrn_s = rrn;
  }
  __syncthreads();
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < q.P) q.p[k] = q.r[k] / sr_precond(q, k) + beta_s * q.p[k];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    q.sc[2 + ((it + 1) & 1)] = rzn_s;
    q.sc[6] = rrn_s;
  }
}

// Converged when r.r <= tol^2 f.f (read after the whole direction launch)
__global__ void __launch_bounds__(64) sr_check_kernel(SrWork q, double tol) {
  if (threadIdx.x == 0 && q.sc[5] == 0.0 && q.sc[6] <= tol * tol * q.sc[1]) q.sc[5] = 1.0;
}

// The vector work of an iteration (sr_sp, sr_update, sr_dir and sr_check above) in
// one launch of one workgroup, for up to kSrVecMaxP columns and 2 MB of slice sums
// (which one compute unit reads): 4 x 256 threads take
// the 256-column blocks four at a time and every sum is formed in those kernels'
// order, so the results are bitwise theirs.  Four launches of some 4.5 us each
// were two thirds of an iteration of a few hundred samples and parameters.  The
// slice sums are read 16 loads at a time: one by one, 32 slices of 4096 columns
// cost more than the launches saved.  200 iterations, with the unrolled loads of
// the products: 200 x 168 5.57 -> 2.94 ms, 1000 x 1400 7.79 -> 5.08, 4096 x 4096
// 16.7 -> 14.3 (32 slices, 1 MB), 4096 x 6000 19.65 -> 18.84 (1.5 MB); with 64 slices
// 8192 x 6144 38.6 -> 42.4 (3 MB), 8192 x 8192 47.5 -> 61.5 (4 MB).
constexpr int kSrVecT = 1024;
constexpr long kSrVecMaxP = 8192, kSrVecMaxSums = 256 * 1024;

// block sums (wave sums in red, blocks of four waves) added in order
__device__ double sr_ordered_sum(const double* red, int nblk) {
  const int lane = threadIdx.x & 63;
  double s = 0.0;
  if (lane < nblk)
    for (int k = 0; k < 4; ++k) s += red[4 * lane + k];
  double t = 0.0;
  for (int b = 0; b < nblk; ++b)
    t += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(s), b),
                          __builtin_amdgcn_readlane(__double2loint(s), b));
  return t;
}

template <int C>
__global__ void __launch_bounds__(kSrVecT) sr_vec_kernel(SrWork q, double* __restrict__ x, int it, double tol) {
  __shared__ double red[3][4 * (kSrVecMaxP / 256)];
  if (q.sc[5] != 0.0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double rzo = q.sc[2 + (it & 1)], ff = q.sc[1];
  double p[C], sp[C], m[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {   // block 4 c + wave / 4
    const long k = tid + (long)kSrVecT * c;
    double pp = 0.0;
    p[c] = sp[c] = 0.0;
    m[c] = 1.0;
    if (k < q.P) {
      double t = 0.0;
#pragma unroll 16
      for (int sl = 0; sl < q.ms; ++sl) t += q.colpart[(long)sl * q.P + k];
      p[c] = q.p[k];
      m[c] = sr_precond(q, k);
      sp[c] = sr_sp(q, k, t, p[c]);
      pp = p[c] * sp[c];
    }
    pp = wave_sum(pp);
    if (lane == 0) red[0][16 * c + wave] = pp;
  }
  __syncthreads();
  const double pSp = sr_ordered_sum(red[0], q.nblk);
  const double alpha = pSp > 0.0 ? rzo / pSp : 0.0;
  double r[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const long k = tid + (long)kSrVecT * c;
    double rz = 0.0, rr = 0.0;
    r[c] = 0.0;
    if (k < q.P) {
      x[k] += alpha * p[c];
      const double rk = q.r[k] - alpha * sp[c];
      q.r[k] = r[c] = rk;
      rz = rk * rk / m[c];
      rr = rk * rk;
    }
    rz = wave_sum(rz);
    rr = wave_sum(rr);
    if (lane == 0) { red[1][16 * c + wave] = rz; red[2][16 * c + wave] = rr; }
  }
  __syncthreads();
  const double rzn = sr_ordered_sum(red[1], q.nblk), rrn = sr_ordered_sum(red[2], q.nblk);
  const double beta = rzo > 0.0 ? rzn / rzo : 0.0;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const long k = tid + (long)kSrVecT * c;
    if (k < q.P) q.p[k] = r[c] / m[c] + beta * p[c];
  }
  if (tid == 0) {
    q.sc[2 + ((it + 1) & 1)] = rzn;
    q.sc[6] = rrn;
    if (rrn <= tol * tol * ff) q.sc[5] = 1.0;
  }
}

__global__ void __launch_bounds__(256) sr_finish_kernel(SrWork q, double* __restrict__ force,
                                                        double* __restrict__ resid) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (force && k < q.P) force[k] = q.f[k];
  if (resid && k == 0) resid[0] = q.sc[1] > 0.0 ? sqrt(q.sc[6] / q.sc[1]) : 0.0;
}

// ---------------------------------------------------------------------------
// One pass over O per iteration (P <= kSrFuseMaxP columns).  The two products of
// an iteration, u = O p and O^T (w o u), read O twice when they are launches of
// their own (2 x 268 MB at 6.1 TB/s for 4096 x 8192: 89 of the 109 us of an
// iteration; four small launches the rest).  Here a workgroup of 1024 threads
// holds all columns (up to 8 a thread): it reads a row, reduces u_i, and adds
// w_i u_i O_i to its columns' sums from the registers the row is in, while the
// next rows are in flight; each workgroup has one contiguous range of samples and
// writes one row of partial sums.  Since every workgroup holds every column it
// also does the vector work of the previous iteration for itself (x, r, beta, p
// and the convergence test, the same bits in each; workgroup 0 writes them),
// under the latency of its first rows, so that an iteration is two launches: this
// one and the sum of the partial rows.
// ---------------------------------------------------------------------------
constexpr int kSrT = 1024;            // threads of the pass
constexpr long kSrFuseMaxP = 8192;    // columns: 8 doubles a thread
constexpr int kSrSlices = 255;        // sample ranges (and one workgroup for Obar . p)
constexpr size_t kSrFuseDoubles = (size_t)2 << 20;   // the fused workspace stays within this

struct SrFused {
  double *r2[2], *p2[2];   // r and p of even and odd iterations
  int S, rows, nsp;        // sample ranges in use, samples a range, workgroups of the sum
  double tol;
};

static long sr_fused_fixed(long P) { return 8 * P + 3 * ((P + 63) / 64) + 16; }

// Sample ranges of the fused pass (0: the two-pass path): as many as the
// workspace bound, the chip and the samples allow, and room for the moments'
// slices.
// Nearly square problems keep the order of sums of the two-pass path: their
// iteration does not converge in 200 steps (the smallest kept singular values of
// O lie near zero) and carries a change of rounding into the step: 1e-9 of it at
// 200 samples x 168 parameters, 1e-5 at 168 x 168 and 300 x 330, where the step
// itself is 1e-8, 5e-4 and 2e-4 from the solution; 1e-12 and less at 200 x 150
// and 207 x 359, which converge in 180 and 140.  The band's lines (3/2 and 3/5 of
// P samples) lie where that was measured, the lower side's with room: 200 x 150
// is inside, 207 x 359 outside.
static bool sr_near_square(int M, long P) { return 2L * M < 3 * P && 3 * P < 5L * M; }

static int sr_fused_slices(int M, long P) {
  if (P > kSrFuseMaxP || sr_near_square(M, P)) return 0;
  long s = ((long)kSrFuseDoubles - sr_fused_fixed(P)) / P;
  s = s < kSrSlices ? s : kSrSlices;
  if (s < 2L * sr_slices(M)) return 0;
  const long rows = (M + s - 1) / s;
  return (int)((M + rows - 1) / rows);
}

static size_t sr_fused_doubles(int M, long P) {
  const long S = sr_fused_slices(M, P), ms2 = 2L * sr_slices(M);
  return S ? (size_t)(sr_fused_fixed(P) + (S > ms2 ? S : ms2) * P) : 0;
}

// sums of two values over the 1024 threads, the same bits in every thread
__device__ double2 blk_sum1024(double a, double b, double (*red)[2][16]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  a = wave_sum(a);
  b = wave_sum(b);
  if (lane == 0) { (*red)[0][wave] = a; (*red)[1][wave] = b; }
  __syncthreads();
  a = (*red)[0][lane & 15];
  b = (*red)[1][lane & 15];
  // (every row of 16 lanes holds the sixteen waves' sums)
  a += dpp_f64<0xB1>(a); a += dpp_f64<0x4E>(a); a += dpp_f64<0x141>(a); a += dpp_f64<0x140>(a);
  b += dpp_f64<0xB1>(b); b += dpp_f64<0x4E>(b); b += dpp_f64<0x141>(b); b += dpp_f64<0x140>(b);
  return double2{a, b};
}

// V columns a load (2: P even and O 16-byte aligned), C loads a row.
template <int V, int C>
__global__ void __launch_bounds__(kSrT)
sr_pass_kernel(SrWork q, SrFused f, const double* __restrict__ O, const double* __restrict__ wts, double* __restrict__ x,
               int it) {
  typedef double vec __attribute__((ext_vector_type(V)));
  __shared__ double red[3][2][16];
  if (q.sc[5] != 0.0) return;   // converged (uniform)
  const int tid = threadIdx.x;
  const bool aux = (int)blockIdx.x == f.S;   // Obar . p
  const int i0 = aux ? 0 : blockIdx.x * f.rows, i1 = aux ? 1 : min(i0 + f.rows, q.M);
  bool ok[C];
  long k0[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    k0[c] = (long)V * (tid + kSrT * c);
    ok[c] = k0[c] < q.P;
  }
  auto load = [&](vec* v, int i) {
    const double* row = aux ? q.Obar : O + (long)i * q.P;
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = ok[c] && i < i1 ? *reinterpret_cast<const vec*>(row + k0[c]) : vec(0.0);
  };
  vec va[C], vb[C], p[C], acc[C];
  load(va, i0);
  load(vb, i0 + 1);
  // the vectors of this iteration
  const int o = it & 1;
  const bool w0 = blockIdx.x == 0;
  if (it == 0) {   // r = f, p = f / m (from the moments); the scalars
    double rz = 0.0, rr = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      p[c] = vec(0.0);
      if (!ok[c]) continue;
      p[c] = *reinterpret_cast<const vec*>(f.p2[0] + k0[c]);
      const vec rk = *reinterpret_cast<const vec*>(f.r2[0] + k0[c]);
#pragma unroll
      for (int v = 0; v < V; ++v) { rz += rk[v] * p[c][v]; rr += rk[v] * rk[v]; }
    }
    const double2 s = blk_sum1024(rz, rr, &red[2]);
    if (w0 && tid == 0) { q.sc[1] = s.y; q.sc[2] = s.x; q.sc[6] = s.y; }
    if (!(s.y > 0.0)) {   // zero force: the step is zero
      if (w0 && tid == 0) q.sc[5] = 1.0;
      return;
    }
  } else {
    const double pSp = blk_sum1024(tid < f.nsp ? q.part1[tid] : 0.0, 0.0, &red[2]).x;
    const double rzo = q.sc[2 + (o ^ 1)];
    const double alpha = pSp > 0.0 ? rzo / pSp : 0.0;
    double rz = 0.0, rr = 0.0;
    vec rn[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      p[c] = vec(0.0);
      rn[c] = vec(0.0);
      if (!ok[c]) continue;
      p[c] = *reinterpret_cast<const vec*>(f.p2[o ^ 1] + k0[c]);
      const vec sp = *reinterpret_cast<const vec*>(q.Sp + k0[c]);
      rn[c] = *reinterpret_cast<const vec*>(f.r2[o ^ 1] + k0[c]) - alpha * sp;
      if (w0) {
#pragma unroll
        for (int v = 0; v < V; ++v) x[k0[c] + v] += alpha * p[c][v];
        *reinterpret_cast<vec*>(f.r2[o] + k0[c]) = rn[c];
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        rz += rn[c][v] * rn[c][v] / sr_precond(q, k0[c] + v);
        rr += rn[c][v] * rn[c][v];
      }
    }
    const double2 s = blk_sum1024(rz, rr, &red[0]);
    if (w0 && tid == 0) { q.sc[2 + o] = s.x; q.sc[6] = s.y; }
    if (s.y <= f.tol * f.tol * q.sc[1]) {   // converged: the same in every workgroup
      if (w0 && tid == 0) q.sc[5] = 1.0;
      return;
    }
    const double beta = rzo > 0.0 ? s.x / rzo : 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if (!ok[c]) continue;
#pragma unroll
      for (int v = 0; v < V; ++v) p[c][v] = rn[c][v] / sr_precond(q, k0[c] + v) + beta * p[c][v];
      if (w0) *reinterpret_cast<vec*>(f.p2[o] + k0[c]) = p[c];
    }
    __syncthreads();   // red[0] is read
  }
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = vec(0.0);
  // two rows at a time, the next two in flight while these reduce
  for (int i = i0; i < i1; i += 2) {
    double ta = 0.0, tb = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int v = 0; v < V; ++v) { ta += va[c][v] * p[c][v]; tb += vb[c][v] * p[c][v]; }
    vec na[C], nb[C];
    load(na, i + 2);
    load(nb, i + 3);
    const double2 u = blk_sum1024(ta, tb, &red[((i - i0) >> 1) & 1]);
    if (aux) {
      if (tid == 0) q.sc[4] = u.x;
      return;
    }
    const double wa = (wts ? wts[i] : 1.0) * u.x, wb = i + 1 < i1 ? (wts ? wts[i + 1] : 1.0) * u.y : 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      acc[c] += wa * va[c] + wb * vb[c];
      va[c] = na[c];
      vb[c] = nb[c];
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (ok[c]) *reinterpret_cast<vec*>(q.colpart + (long)blockIdx.x * q.P + k0[c]) = acc[c];
}

// S'p from the partial rows, and partial sums of p . S'p: 64 columns a workgroup,
// wave g the rows g, g + 16, ...
__global__ void __launch_bounds__(kSrT) sr_pass_sum_kernel(SrWork q, SrFused f, int it) {
  __shared__ double part[16][64];
  if (q.sc[5] != 0.0) return;
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const long k = (long)blockIdx.x * 64 + lane;
  double t = 0.0;
  if (k < q.P) {
#pragma unroll 8
    for (int s = g; s < f.S; s += 16) t += q.colpart[(long)s * q.P + k];
  }
  part[g][lane] = t;
  __syncthreads();
  if (g) return;
  double pp = 0.0;
  if (k < q.P) {
    for (int s = 1; s < 16; ++s) t += part[s][lane];
    const double pk = f.p2[it & 1][k];
    const double sp = sr_sp(q, k, t, pk);
    q.Sp[k] = sp;
    pp = pk * sp;
  }
  pp = wave_sum(pp);
  if (lane == 0) q.part1[blockIdx.x] = pp;
}

// The last iteration's step (none with its = 0) and the outputs: one workgroup.
__global__ void __launch_bounds__(kSrT) sr_pass_last_kernel(SrWork q, SrFused f, double* __restrict__ x,
                                                           double* __restrict__ force, double* __restrict__ resid,
                                                           int its) {
  __shared__ double red[2][2][16];
  const int tid = threadIdx.x, o = (its - 1) & 1;
  const bool open = q.sc[5] == 0.0;   // not converged (read by all before any write)
  double ff = q.sc[1], rr = q.sc[6], alpha = 0.0;
  if (open && its > 0) {
    const double pSp = blk_sum1024(tid < f.nsp ? q.part1[tid] : 0.0, 0.0, &red[0]).x;
    alpha = pSp > 0.0 ? q.sc[2 + o] / pSp : 0.0;
  }
  double s = 0.0;
  for (long k = tid; k < q.P; k += kSrT) {
    if (force) force[k] = q.f[k];
    if (its == 0) s += q.f[k] * q.f[k];
    else if (open) {
      x[k] += alpha * f.p2[o][k];
      const double rk = f.r2[o][k] - alpha * q.Sp[k];
      s += rk * rk;
    }
  }
  s = blk_sum1024(s, 0.0, &red[1]).x;
  if (its == 0) ff = rr = s;
  else if (open) rr = s;
  if (tid == 0 && resid) resid[0] = ff > 0.0 ? sqrt(rr / ff) : 0.0;
}

size_t sr_workspace_min(int M, long P) {
  const long nblk = (P + 255) / 256;
  return (size_t)(6 * P + M + 3 * nblk + 16 + 2L * sr_slices(M) * P);
}

size_t sr_workspace_doubles(int M, long P) {
  const size_t a = sr_workspace_min(M, P), b = sr_fused_doubles(M, P);
  return a > b ? a : b;
}

// the moments of the samples: Obar, the diagonal of S, the force; r = f, p = f / m
static hipError_t sr_moments(const SrWork& q, const double* O, const double* el, const double* wts, double* delta,
                             hipStream_t st) {
  const dim3 gk(q.nblk), g2(q.nblk, q.ms), blk(256);
  hipLaunchKernelGGL(sr_wsum_kernel, dim3(1), blk, 0, st, q, wts);
  hipLaunchKernelGGL(sr_colsum_kernel, g2, blk, 0, st, q, O, el, wts, 0);
  hipLaunchKernelGGL(sr_mean_kernel, gk, blk, 0, st, q);
  hipLaunchKernelGGL(sr_colsum_kernel, g2, blk, 0, st, q, O, el, wts, 1);
  hipLaunchKernelGGL(sr_moments_kernel, gk, blk, 0, st, q, delta);
  hipLaunchKernelGGL(sr_init_kernel, dim3(1), dim3(64), 0, st, q);
  return hipGetLastError();
}

hipError_t launch_sr_step(int M, long P, const double* O, const double* el, const double* wts, double eps,
                          int max_iter, double tol, double* delta, double* force, double* resid, double* work,
                          size_t work_doubles, hipStream_t st) {
  SrWork q;
  q.P = P; q.M = M; q.nblk = (int)((P + 255) / 256); q.eps = eps;
  q.ms = sr_slices(M); q.rows = (M + q.ms - 1) / q.ms;
  const dim3 gk(q.nblk), g2(q.nblk, q.ms), blk(256);
  const int S = sr_fused_slices(M, P);
  if (S > 0 && work_doubles >= sr_fused_doubles(M, P)) {
    SrFused f;
    f.S = S; f.rows = (M + S - 1) / S; f.nsp = (int)((P + 63) / 64); f.tol = tol;
    double* p = work;   // (pairs of columns: the vectors of length P first, 16-byte aligned when P is even)
    q.Obar = p; p += P; q.d = p; p += P; q.f = p; p += P; q.Sp = p; p += P;
    f.r2[0] = p; p += P; f.r2[1] = p; p += P; f.p2[0] = p; p += P; f.p2[1] = p; p += P;
    q.r = f.r2[0]; q.p = f.p2[0]; q.u = nullptr;
    q.colpart = p; p += (S > 2 * q.ms ? (long)S : 2L * q.ms) * P;
    q.part1 = p; p += f.nsp; q.part2 = p; p += f.nsp; q.part3 = p; p += f.nsp;
    q.sc = p;
    hipError_t e = sr_moments(q, O, el, wts, delta, st);
    if (e != hipSuccess) return e;
    e = hipSuccess;
    const bool pair = P % 2 == 0 && ((uintptr_t)O | (uintptr_t)work | (uintptr_t)delta) % 16 == 0;
    const int per = (int)((P + kSrT - 1) / kSrT);
    for (int it = 0; it < max_iter; ++it) {
#define QMC_SR(V, C) hipLaunchKernelGGL((sr_pass_kernel<V, C>), dim3(S + 1), dim3(kSrT), 0, st, q, f, O, wts, delta, it)
      if (pair) {
        if (per <= 2) QMC_SR(2, 1);
        else if (per <= 4) QMC_SR(2, 2);
        else if (per <= 6) QMC_SR(2, 3);
        else QMC_SR(2, 4);
      } else {
        if (per <= 1) QMC_SR(1, 1);
        else if (per <= 2) QMC_SR(1, 2);
        else if (per <= 4) QMC_SR(1, 4);
        else QMC_SR(1, 8);
      }
#undef QMC_SR
      hipLaunchKernelGGL(sr_pass_sum_kernel, dim3(f.nsp), dim3(kSrT), 0, st, q, f, it);
    }
    hipLaunchKernelGGL(sr_pass_last_kernel, dim3(1), dim3(kSrT), 0, st, q, f, delta, force, resid, max_iter);
    return hipGetLastError();
  }
  double* p = work;
  q.Obar = p; p += P; q.d = p; p += P; q.f = p; p += P; q.r = p; p += P; q.p = p; p += P; q.Sp = p; p += P;
  q.u = p; p += M; q.part1 = p; p += q.nblk; q.part2 = p; p += q.nblk; q.part3 = p; p += q.nblk;
  q.colpart = p; p += 2L * q.ms * P; q.sc = p;
  const hipError_t e = sr_moments(q, O, el, wts, delta, st);
  if (e != hipSuccess) return e;
  for (int it = 0; it < max_iter; ++it) {
    hipLaunchKernelGGL(sr_op_kernel, dim3(M + 1), blk, 0, st, q, O);
    hipLaunchKernelGGL(sr_colsum_kernel, g2, blk, 0, st, q, O, el, wts, 2);
    if (P <= kSrVecMaxP && q.ms * P <= kSrVecMaxSums) {
      const int per = (int)((P + kSrVecT - 1) / kSrVecT);
      if (per <= 1) hipLaunchKernelGGL(sr_vec_kernel<1>, dim3(1), dim3(kSrVecT), 0, st, q, delta, it, tol);
      else if (per <= 2) hipLaunchKernelGGL(sr_vec_kernel<2>, dim3(1), dim3(kSrVecT), 0, st, q, delta, it, tol);
      else if (per <= 4) hipLaunchKernelGGL(sr_vec_kernel<4>, dim3(1), dim3(kSrVecT), 0, st, q, delta, it, tol);
      else hipLaunchKernelGGL(sr_vec_kernel<8>, dim3(1), dim3(kSrVecT), 0, st, q, delta, it, tol);
      continue;
    }
    hipLaunchKernelGGL(sr_sp_kernel, gk, blk, 0, st, q);
    hipLaunchKernelGGL(sr_update_kernel, gk, blk, 0, st, q, delta, it);
    hipLaunchKernelGGL(sr_dir_kernel, gk, blk, 0, st, q, it);
    hipLaunchKernelGGL(sr_check_kernel, dim3(1), dim3(64), 0, st, q, tol);
  }
  hipLaunchKernelGGL(sr_finish_kernel, gk, blk, 0, st, q, force, resid);
  return hipGetLastError();
}

}  // namespace qmc

// ---------------------------------------------------------------------------
// SR step without allocation: the workspace is a fixed device array of the
// library (one copy per GPU, alive until the process ends).  Host code never
// passes the array's name to a kernel or a copy: on the host that name is a
// stand-in, not a device address.  Its address on each device is looked up
// once, with that device current, and kept.
// ---------------------------------------------------------------------------
constexpr size_t kSrStaticDoubles = (size_t)2 << 20;   // 16 MiB of FP64
static __device__ __align__(256) double scratch[kSrStaticDoubles];
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

extern "C" qmc_status qmc_sr_step_static(int32_t n_samples, int64_t n_params, const double* O, const double* e_loc,
                                         const double* weights, double eps, int32_t max_iter, double tol,
                                         double* delta, double* force, double* residual, hipStream_t stream) {
  using namespace qmc;
  if (!O || !e_loc || !delta) return set_error(QMC_ERR_ARG, "null argument");
  if (n_samples <= 0 || n_params <= 0 || max_iter < 0) return set_error(QMC_ERR_ARG, "bad sizes");
  if (!(eps >= 0.0) || !(tol >= 0.0)) return set_error(QMC_ERR_ARG, "eps and tol must be >= 0");
  if (sr_workspace_min(n_samples, (long)n_params) > kSrStaticDoubles)
    return set_error(QMC_ERR_SHAPE, "SR problem needs more than the 16 MiB static workspace "
                                    "(qmc_sr_workspace_size > 16777216 bytes): use qmc_sr_step");
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return set_error(QMC_ERR_HIP, hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return set_error(QMC_ERR_UNSUPPORTED, "device ordinal beyond 63");
  double* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p) return set_error(QMC_ERR_HIP, "hipGetSymbolAddress of the SR scratch failed");
      g_scratch_ptr[dev] = (double*)p;
    }
    ptr = g_scratch_ptr[dev];
  }
  e = launch_sr_step(n_samples, (long)n_params, O, e_loc, weights, eps, max_iter, tol, delta, force, residual, ptr,
                     kSrStaticDoubles, stream);
  if (e != hipSuccess) return set_error(QMC_ERR_HIP, hipGetErrorString(e));
  return QMC_OK;
}
