// Device code shared by the resident moves (chain.hip) and the evaluation of small
// systems (small_eval.hip): the inverse of a matrix in LDS by one workgroup of
// 256 threads.
#pragma once

#include "internal.h"

namespace qmc {

constexpr int kChainT = 256;               // threads
constexpr int kChainSmallN = 64;           // rows of W that one workgroup inverts: a lane each

// leading dimension of B: even (column pairs), and a column's entries over
// different banks
__host__ __device__ inline int chain_ld(int n) { return (n + 1) / 2 * 2 + 2; }

// threadIdx.x through an opaque move: what is computed from it stays in the
// phase that uses it instead of being held in registers over the move loop.
__device__ __forceinline__ int chain_tid() {
  int z;
  asm volatile("v_mov_b32 %0, 0" : "=v"(z));
  return (int)threadIdx.x + z;
}

// The last step of chain_invert: inverse element (i, p_c) = T[p_i][c] / pivot_i.
template <int NQ>
__device__ __forceinline__ void chain_permute(double* B, int n, int ld, int tid, bool tr, const double* ip, const int* prow) {
  double t[NQ];
  int at[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int x = tid + kChainT * q, i = x / n, c = x - i * n;
    at[q] = -1;
    if (x < n * n) {
      t[q] = B[prow[i] * ld + c] * ip[i];
      at[q] = tr ? prow[c] * ld + i : i * ld + prow[c];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    if (at[q] >= 0) B[at[q]] = t[q];
}

// B[n][ld] (LDS) <- its inverse, in place: Gauss-Jordan with the pivot of step k
// the largest |entry| of column k among the rows not yet pivoted (lowest row on
// ties), n <= 64.  Thread (g, j) keeps column j of rows g, g + G, ...; the step
// publishes the next pivot column as it updates it, every wave finds the pivot
// for itself, and a pivot row is left unscaled until the end (only its column-k
// entry becomes 1), so a step takes one barrier.  Afterwards element (p_k, k')
// over pivot k is inverse element (k, p_k'), put in place by the last step
// (transposed when tr).  log|det| and sign to wave 0; singular: returns true and
// B is not a number.  Pivots, multipliers, updates and the order of the
// logarithms are the row kernel's: the results are bitwise its.
__device__ bool chain_invert(double* B, int n, int ld, bool tr, double* fc, double* ips, int* prow, double& logdet,
                             double& sign) {
  const int tid = chain_tid(), lane = tid & 63;
  const int G = min(kChainT / n, 16), g = tid / n, j = tid - g * n;
  bool used = lane >= n;
  double own = 1.0, step_ip = 1.0;   // this row's pivot; step `lane`'s pivot inverted
  int step_p = lane, own_k = lane;   // the row pivoted at step `lane`; the step that pivoted this row
  if (tid < n) fc[tid] = B[tid * ld];
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    const double* f = fc + 64 * (k & 1);
    double* fn = fc + 64 * ((k + 1) & 1);
    const double fl = lane < n ? f[lane] : 0.0;
    const unsigned long long key =
        used ? 0ull : ((__double_as_longlong(fabs(fl)) & ~0xFFull) | (unsigned long long)(255 - lane));
    const unsigned long long best = wave_max_u64(key);
    const int p = 255 - (int)(best & 0xFFull);
    const double piv = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(fl), p & 63),
                                        __builtin_amdgcn_readlane(__double2loint(fl), p & 63));
    if (!(piv != 0.0)) {   // the same for every wave
      __syncthreads();
      const double nanv = __longlong_as_double(0x7ff8000000000000LL);
      for (int q = tid; q < n * ld; q += kChainT) B[q] = nanv;
      __syncthreads();
      logdet = -__builtin_inf();
      sign = 0.0;
      return true;
    }
    const double ip = 1.0 / piv;
    if (lane == p) { used = true; own = piv; own_k = k; }
    if (lane == k) { step_ip = ip; step_p = p; }
    if (g < G) {
      const double pr = B[p * ld + j];
      for (int i = g; i < n; i += G) {
        double v = pr;
        if (i == p) {
          if (j == k) B[i * ld + j] = 1.0;
        } else {
          const double gi = f[i] * ip;
          v = j == k ? -gi : fma(-gi, pr, B[i * ld + j]);
          B[i * ld + j] = v;
        }
        if (j == k + 1) fn[i] = v;
      }
    }
    __syncthreads();
  }
  if (tid < n) { prow[tid] = step_p; ips[tid] = step_ip; }   // wave 0's lanes
  __syncthreads();
  if (n <= 16) chain_permute<1>(B, n, ld, tid, tr, ips, prow);
  else if (n <= 32) chain_permute<4>(B, n, ld, tid, tr, ips, prow);
  else chain_permute<16>(B, n, ld, tid, tr, ips, prow);
  if (tid < 64) {
    // the parity of the pivot permutation by counting inversions, and the pivots' signs
    int odd = __popcll(__ballot(lane < n && own < 0.0));
    for (int i = 0; i + 1 < n; ++i) {
      const int ki = __builtin_amdgcn_readlane(own_k, i);
      odd += __popcll(__ballot(lane > i && lane < n && own_k < ki));
    }
    logdet = wave_sum(lane < n ? log(fabs(own)) : 0.0);
    sign = (odd & 1) ? -1.0 : 1.0;
  }
  __syncthreads();
  return false;
}

}  // namespace qmc
