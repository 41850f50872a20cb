// Evaluation of a small system in one launch: a workgroup of 256 threads takes a
// walker from its positions to the row dots (basis values, P, W, W^{-1} and
// log|det|, the cofactor rows, grad and lap of the determinant), with the walker's
// rows in LDS.
//
// What bounds these evaluations is their launches: 14 kernels of 2 to 7 us and
// three copies for 64 walkers x 10 e, L = 24 (58 us of kernels in 69 us, the
// arithmetic under 2 us); this kernel and the Jastrow's take 20.5 us.  Every product runs on the FP64 matrix cores in the k order of the
// batched kernels and the inverse is theirs step by step, so the results are
// bitwise those of the batched path.
#include "internal.h"
#include "resident_dev.h"
#include <algorithm>

namespace qmc {

constexpr int kSmallEvalLds = 80 * 1024;   // two workgroups per compute unit

struct SmallLayout { int phi, P, B, fc, ips, prow, r, total; };

static SmallLayout small_layout(const SysDev& s) {
  SmallLayout o{};
  const int ldp = s.Lp + 2;
  int at = 0;
  auto take = [&](int& p, int bytes) { p = at; at += (bytes + 15) / 16 * 16; };
  take(o.phi, 8 * s.N * ldp);
  take(o.P, 8 * std::max(s.N * ldp, 4 * s.Lq));   // (and a wave's primitives each)
  take(o.B, 8 * s.nu * chain_ld(s.nu));
  take(o.fc, 8 * 2 * kChainSmallN);
  take(o.ips, 8 * kChainSmallN);
  take(o.prow, 4 * kChainSmallN);
  take(o.r, 8 * 3 * s.N);
  o.total = at;
  return o;
}

typedef double sdx4 __attribute__((ext_vector_type(4)));

// Rows in LDS are padded by two doubles: the 16 x 4 operand reads of a matrix
// tile then touch every bank once.
__global__ void __launch_bounds__(kChainT, 2) small_eval_kernel(SysDev s, WalkDev w, const double* r_in,
                                                                SmallLayout ly) {
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wk = blockIdx.x;
  const int li = lane & 15, lk = lane >> 4;
  const int N = s.N, n = s.nu, nd = s.nd, nk = s.nk, L = s.L, Lp = s.Lp, ldp = Lp + 2, ld = chain_ld(n);
  double *phi = (double*)(lds + ly.phi), *P = (double*)(lds + ly.P), *B = (double*)(lds + ly.B),
         *fc = (double*)(lds + ly.fc), *ips = (double*)(lds + ly.ips), *r = (double*)(lds + ly.r);
  int* prow = (int*)(lds + ly.prow);
  const long row0 = (long)wk * N;
  for (int q = tid; q < 3 * N; q += kChainT) {
    const double x = r_in[row0 * 3 + q];
    r[q] = x;
    w.r[row0 * 3 + q] = x;
    w.rpos_P[row0 * 3 + q] = x;   // every P row is built here
  }
  __syncthreads();
  // basis values
  double* phig = (double*)w.phi + row0 * Lp;
  if (s.Lq == 0) {
    for (int q = tid; q < N * Lp; q += kChainT) {
      const int i = q / Lp, mu = q - i * Lp;
      const double v = mu < L ? basis_value(s, mu, r[3 * i], r[3 * i + 1], r[3 * i + 2]) : 0.0;
      phi[i * ldp + mu] = v;
      phig[q] = v;
    }
  } else {   // contracted: a wave takes rows, their primitives in P's place
    double* qv = P + wave * s.Lq;
    for (int i = wave; i < N; i += 4) {
      __builtin_amdgcn_wave_barrier();
      for (int mu = lane; mu < s.Lq; mu += 64) qv[mu] = basis_value(s, mu, r[3 * i], r[3 * i + 1], r[3 * i + 2]);
      __builtin_amdgcn_wave_barrier();
      for (int c = lane; c < Lp; c += 64) {
        double v = 0.0;
        if (c < L)
          for (int k = s.con_ptr[c]; k < s.con_ptr[c + 1]; ++k) v += s.con_coef[k] * qv[s.con_idx[k]];
        phi[i * ldp + c] = v;
        phig[i * Lp + c] = v;
      }
    }
  }
  __syncthreads();
  // P: a wave takes column tiles of one half, all its row tiles together (Lambda's
  // rows come from L2 once)
  double* Pg = (double*)w.P + row0 * Lp;
  const int CT = Lp / 16;
  for (int it = wave; it < 2 * CT; it += 4) {
    const int h = it / CT, ct = it - h * CT;
    const int m = h == 0 ? n : nd, i0 = h == 0 ? 0 : n, RT = (m + 15) / 16;
    const double* lc = (h == 0 ? s.lam : s.lamT) + (long)lk * Lp + ct * 16 + li;
    sdx4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = sdx4{0.0, 0.0, 0.0, 0.0};
    int ar[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) ar[t] = (i0 + min(16 * t + li, m - 1)) * ldp + lk;   // (rows past m: discarded)
    double b[4], bn[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = lc[(long)(4 * u) * Lp];
    for (int k = 0; k < Lp; k += 16) {
      const bool more = k + 16 < Lp;
#pragma unroll
      for (int u = 0; u < 4; ++u) bn[u] = more ? lc[(long)(k + 16 + 4 * u) * Lp] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (t < RT) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(phi[ar[t] + k + 4 * u], b[u], acc[t], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) b[u] = bn[u];
    }
    // lane holds column lane % 16 and rows 4 r + lane / 16
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 16 * t + 4 * q + lk;
        if (i < m) {
          P[(i0 + i) * ldp + ct * 16 + li] = acc[t][q];
          Pg[(long)(i0 + i) * Lp + ct * 16 + li] = acc[t][q];
        }
      }
  }
  __syncthreads();
  // W = [P_up Phi_dn^T | Phi_up U]
  double* Wg = w.W + (long)wk * n * n;
  {
    const int RT = (n + 15) / 16, PT = (nd + 15) / 16, UT = (nk + 15) / 16;
    for (int it = wave; it < RT * (PT + UT); it += 4) {
      const int rt = it / (PT + UT), ct = it - rt * (PT + UT);
      const bool un = ct >= PT;
      const int c = (un ? (ct - PT) : ct) * 16 + li, cn = un ? nk : nd;
      const double* a = (un ? phi : P) + min(16 * rt + li, n - 1) * ldp + lk;
      const double* bl = phi + (n + min(c, nd - 1)) * ldp + lk;
      const double* bu = un ? s.Uph + (long)min(c, nk - 1) * Lp + lk : nullptr;
      sdx4 acc = sdx4{0.0, 0.0, 0.0, 0.0};
      if (un)
        for (int k = 0; k < Lp; k += 4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k], bu[k], acc, 0, 0, 0);
      else
        for (int k = 0; k < Lp; k += 16)
#pragma unroll
          for (int u = 0; u < 16; u += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k + u], bl[k + u], acc, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 16 * rt + 4 * q + lk, j = (un ? nd : 0) + c;
        if (i < n && c < cn) {
          B[i * ld + j] = acc[q];
          Wg[(long)i * n + j] = acc[q];
        }
      }
    }
  }
  __syncthreads();
  double ldet = 0.0, sdet = 0.0;
  const bool sing = chain_invert(B, n, ld, false, fc, ips, prow, ldet, sdet);
  if (tid == 0) {
    w.logdet[wk] = ldet;
    w.detsign[wk] = sdet;
    w.singular[wk] = sing ? 1 : 0;
  }
  for (int q = tid; q < n * n; q += kChainT) {
    const int i = q / n, k = q - i * n;
    w.A[(long)wk * n * n + q] = B[i * ld + k];
  }
  // cofactor rows, into phi's place too:
  //   Yt_up[i] = sum_j A[j][i] P_dn[j] (+ the unpaired orbitals'), Yt_dn[j] = sum_i A[j][i] P_up[i]
  double* Yg = w.Yt + row0 * Lp;
  for (int it = wave; it < 2 * CT; it += 4) {
    const int h = it / CT, ct = it - h * CT;
    const int m = h == 0 ? n : nd, kk = h == 0 ? nd : n;
    const int RT = (m + 15) / 16;
    for (int rt = 0; rt < RT; ++rt) {
      const int i = min(16 * rt + li, m - 1);
      sdx4 acc = sdx4{0.0, 0.0, 0.0, 0.0};
      for (int k = 0; k < kk; k += 4) {
        const int j = min(k + lk, kk - 1);
        const double av = h == 0 ? B[j * ld + i] : B[i * ld + j];
        const double a = k + lk < kk ? av : 0.0;
        const double b = k + lk < kk ? P[((h == 0 ? n : 0) + j) * ldp + ct * 16 + li] : 0.0;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
      }
      sdx4 acu = sdx4{0.0, 0.0, 0.0, 0.0};
      if (h == 0 && nk > 0)
        for (int k = 0; k < nk; k += 4) {
          const int l = min(k + lk, nk - 1);
          const double a = k + lk < nk ? B[(nd + l) * ld + i] : 0.0;
          const double b = k + lk < nk ? s.Uph[(long)l * Lp + ct * 16 + li] : 0.0;
          acu = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acu, 0, 0, 0);
        }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int io = 16 * rt + 4 * q + lk;
        if (io < m) {
          const double v = h == 0 && nk > 0 ? acc[q] + acu[q] : acc[q];
          const int row = (h == 0 ? 0 : n) + io;
          phi[row * ldp + ct * 16 + li] = v;
          Yg[(long)row * Lp + ct * 16 + li] = v;
        }
      }
    }
  }
  __syncthreads();
  // row dots (one wave per row, as the batched kernel's)
  for (int i = wave; i < N; i += 4) {
    const double px = r[3 * i], py = r[3 * i + 1], pz = r[3 * i + 2];
    const double* y = phi + i * ldp;
    double sx = 0.0, sy = 0.0, sz = 0.0, sl = 0.0;
    for (int mu = lane; mu < s.nprim(); mu += 64) {
      double v, gx, gy, gz, lp;
      basis_vgl(s, mu, px, py, pz, v, gx, gy, gz, lp);
      const double yy = s.Lq ? prim_weight(s, mu, y) : y[mu];
      sx += gx * yy; sy += gy * yy; sz += gz * yy; sl += lp * yy;
    }
    const double sum = wave_sum4(sx, sz, sy, sl);
    if ((lane & 15) == 0) w.D[(row0 + i) * 4 + (lane >> 4)] = sum;
  }
}

// Systems the one-launch evaluation takes: FP64, W of at most 64 rows and a
// walker's rows within 80 KiB of LDS, where it is the faster path (batched ->
// one launch, us an evaluation):
//   L = 25, 10 e    64 walkers 61 -> 22, 1024 88 -> 42, 16384 667 -> 528
//   L = 60, 24 e    64 walkers 63 -> 34, 1024 114 -> 73, 16384 966 -> 890
//   L = 96, 32 e    64 walkers 62 -> 52, 512 94 -> 71, 1024 126 -> 132, 4096 351 -> 488
//   L = 156, 12 e   64 walkers 62 -> 55, 512 87 -> 73, 1024 121 -> 131
//   L = 256, 7 e    64 walkers 74 -> 105 (a walker's share of Lambda from L2 is all of it)
//   L = 60 of 300 primitives, 31 e   64 walkers 86 -> 95 (basis values and row dots by one workgroup)
//   L = 64, 32 e    512 walkers 88 -> 55, 4096 311 -> 287, 16384 1122 -> 1116
//   L = 50, 40 e    1024 walkers 144 -> 121, 4096 395 -> 394, 16384 1381 -> 1509
//   L = 48, 48 e    512 walkers 119 -> 89, 768 144 -> 146, 2048 281 -> 327, 16384 1825 -> 2510
//   L = 64, 64 e    512 walkers 146 -> 121, 768 178 -> 199, 16384 2526 -> 3463
// Past 512 walkers (two a compute unit) the batched kernels' many waves hide
// what two workgroups cannot, unless the launches still outweigh it: up to L = 64
// at any number of walkers with 16 rows of W, up to 4096 walkers with 20 (one
// workgroup's inverse and row dots grow with the rows).
bool small_eval_ok(const SysDev& s, const WalkDev& w) {
  return s.precision == QMC_FP64 && !s.pairing && w.rpos_P && s.nu >= 1 && s.nd >= 1 && s.nu <= kChainSmallN &&
         s.Lp % 32 == 0 && s.Lp <= 160 && s.nprim() <= 256 &&
         (w.Wk <= 512 || (s.Lp <= 64 && (s.nu <= 16 || (s.nu <= 20 && w.Wk <= 4096)))) &&
         small_layout(s).total <= kSmallEvalLds;
}

hipError_t launch_small_eval(const SysDev& s, const WalkDev& w, const double* r, hipStream_t st) {
  if (!small_eval_ok(s, w)) return hipErrorInvalidValue;
  const SmallLayout ly = small_layout(s);
  hipLaunchKernelGGL(small_eval_kernel, dim3(w.Wk), dim3(kChainT), ly.total, st, s, w, r, ly);
  return hipGetLastError();
}

}  // namespace qmc
