// Resident moves: one workgroup per walker makes a run of Metropolis moves with
// the walker's moving state in LDS.
//
// What bounds the moves is latency and, for large walker sets, the stream of P.
// With a launch per phase a move of 20 electrons was some thirty dependent trips
// to memory (25.7 us a move at 256 walkers x 20 e, L = 44 with a Jastrow basis;
// the arithmetic of a move is well under 1 us).  A run in one launch that staged
// the delayed-update buffers anew for every move took 36 us a move at 1024
// walkers x 160 e, 27 us at 256 walkers x 256 e (one workgroup per compute unit,
// waiting on its own dependent steps).  Nothing in a move leaves its walker, so
// here a workgroup holds in LDS
//   the inverse itself in the orientation of the moving spin, B = W^{-1} for up
//   moves, its transpose for down moves: both spins read column e and update by
//   the same Sherman-Morrison step
//     R = sum_j w_j B[j][e],  B[j][k] -= B[j][e] (sum_i w_i B[i][k] - delta_ek) / R,
//   a column read and an n x n update in place of the chains of dependent
//   products of the delayed form;
//   positions, nuclei, the sums over the Jastrow basis and the draws of 32 steps.
// A wave computes psi(r') of its own basis functions, lists those it keeps and
// streams their columns of the transposed P rows without waiting for the other
// waves; the waves meet once for a rejected move (the sums of w and of the
// Jastrow change; eight waves once more) and twice more for an accepted one.  Columns are read a row
// pair a lane, several functions a load where n is small, 12 loads in flight.
//
// Two forms, chosen by size (chain_class):
//   small   (W of at most 64 rows, a half of P in LDS, 80 KiB in all): the
//           refreshes, changes of spin and P rebuilds run in the kernel too, so
//           any number of moves is one launch; every function is streamed (from
//           LDS, where screening would cost more than it saves).
//   large   (W of at most 128 rows; 512 threads where one workgroup fills a compute
//           unit, chain_threads): the transposed rows stay in global memory
//           and are screened (where the kept functions give a small ratio, those
//           that matter beside it are streamed too); a launch ends where the schedule refreshes or
//           changes spin.  Walkers past two (n <= 90) or one per compute unit
//           wait for the first ones to finish their run, which keeps the rows in
//           use within the 256 MB last-level cache.  Single proposals of these
//           systems are the same code with one move, and single accepts its update a
//           few columns a workgroup (bitwise a run's).
// The Jastrow basis rows and their matrix are in LDS too in the small form; in the
// large form they stay in global memory (a move reads one row of each ahead of
// its use, an accept a block of the matrix from L2), where they kept systems out:
// 149 walkers x 76 e, 152 Jastrow functions 84.9 -> 33.0 us a move, 1024 x 128 e,
// 256 functions 604 -> 134.
// Contracted orbitals take the same two forms: the primitives at r' go to LDS and
// the waves meet once more, then each wave combines its own orbitals.
// W's row or column and the basis row (and in the small form P's rows) go to the
// walker's arrays in global memory; at the end they hold the usual state with an
// empty delayed-update buffer.  The schedule is that of the per-move path.
#include <hip/hip_ext.h>

#include "internal.h"
#include "resident_dev.h"
#include <algorithm>

namespace qmc {

constexpr int kChainMaxN = 128;            // rows of W: two a lane
constexpr int kChainDraws = 32;            // steps whose draws are staged together
constexpr int kChainU = 12;                // column loads in flight per wave
constexpr int kChainG = 8;                 // row groups of an n x n pass
constexpr int kChainLogs = 32;             // accepted moves whose logarithms are taken together
constexpr int kChainSmallLds = 80 * 1024;  // two workgroups per compute unit
constexpr int kChainMaxLds = 160 * 1024;

static int chain_groups(int n, int T) { return std::min(T / ((n + 1) / 2), kChainG); }

struct ChainLayout {   // byte offsets in LDS
  int qv, cc, ci, cp, area, B, lv, lm, r, nuc, draw, red, part, ws, cs, lg, list, prow, chi, hv, G, jm, chin, jb, jk, M3, total;
};

struct ChainArgs {
  int e0, steps;            // first electron, moves
  int cap;                  // attempts of one spin between refreshes
  int since0, buf_spin0;    // schedule state at the start
  int valid0;               // P halves that hold (bit 0 up, 1 down)
  int all_rows;             // rebuild every row of a half, not only the moved ones
  int store_A;              // write the inverse back (0: a refresh follows)
  const double* Ainv;       // [Wk][n][n] the inverse at the start
  const double* disp;       // [steps][Wk][3] (propose: null)
  const double* unif;       // [steps][Wk]
  const double* r_new;      // propose: [Wk][3], or null and disp
  double* ratio_out;        // propose: [Wk] or null
  int32_t* cnt;             // [Wk] or null
  int groups, pst;          // row groups of an n x n pass; from one move's partial sums to the next's
  int area_bytes, cw, lsh, nuc_lds;   // P area, list entries a wave, log2 of the lanes a column takes, nuclei in LDS
  int con_lds;              // the contraction coefficients in LDS
  ChainLayout ly;
};

// propose: a single proposal (which reads the one column of the inverse it needs)
static ChainLayout chain_layout(const SysDev& s, bool small, ChainArgs& a, bool propose = false, int T = kChainT) {
  ChainLayout o{};
  const int n = s.nu, ld = chain_ld(n), f8 = 8;
  a.area_bytes = small ? f8 * std::max(s.ptn * s.Lp, 16 * (s.Lp + 2)) : 0;
  const int W = T / 64;   // waves
  a.cw = 64 * (small && s.Lq > 0 ? 2 : (s.L + T - 1) / T);   // (the kernel's QL)
  a.lsh = 2;
  while ((2 << a.lsh) < s.ptn) ++a.lsh;
  int at = 0;
  auto take = [&](int& p, int bytes) { p = at; at += (bytes + 15) / 16 * 16; };
  take(o.area, a.area_bytes);
  if (!propose) take(o.B, f8 * n * ld);
  take(o.lv, f8 * W * a.cw);
  take(o.lm, 2 * W * a.cw);
  take(o.r, f8 * 3 * s.N);
  take(o.draw, f8 * 4 * kChainDraws);
  take(o.red, f8 * (2 * W + 8));   // partial sums of two moves, the two-body parameters
  a.groups = chain_groups(n, T);
  const int sums = std::max(W, a.groups) * s.ptn;
  a.pst = W == 4 ? sums : 0;   // (eight waves: one buffer)
  take(o.part, f8 * std::max(sums + a.pst, 2 * kChainSmallN));   // (and two pivot columns of a refresh)
  take(o.ws, f8 * (n + 1));
  take(o.cs, f8 * (n + 1));
  take(o.lg, f8 * 2 * kChainLogs);
  take(o.prow, 4 * (small ? kChainSmallN : W));
  if (small) take(o.list, 4 * (kChainSmallN + 1));
  if (s.LJ > 0) {
    if (small) {   // (large form: in global memory)
      take(o.chi, f8 * s.N * s.LJ);
      take(o.hv, f8 * s.N * s.LJ);
      take(o.M3, f8 * 2 * s.LJ * (2 * s.LJ + 1));
    }
    take(o.G, f8 * 2 * s.LJ);
    take(o.jm, f8 * 2 * s.LJ);
    take(o.chin, f8 * s.LJ);
    take(o.jb, f8 * 4 * s.LJ);
    take(o.jk, 4 * s.LJ);
  }
  if (s.Lq > 0) take(o.qv, f8 * s.Lq);
  // the nuclei and the contraction last: a system that only just fits reads them
  // from global memory
  a.nuc_lds = at + f8 * 5 * s.n_nuc <= kChainMaxLds ? 1 : 0;
  if (a.nuc_lds) take(o.nuc, f8 * 5 * s.n_nuc);
  a.con_lds = s.Lq > 0 && at + 10 * s.nnz_con + 4 * (s.L + 1) + 48 <= (small ? kChainSmallLds : kChainMaxLds) ? 1 : 0;
  if (a.con_lds) {
    take(o.cc, f8 * s.nnz_con);
    take(o.cp, 4 * (s.L + 1));
    take(o.ci, 2 * s.nnz_con);
  }
  o.total = at;
  return o;
}
static_assert(kChainLogs <= 64, "one lane a logarithm");

typedef double cdx4 __attribute__((ext_vector_type(4)));

// The P rows of half h whose electron has moved since they were built (all of
// them with `all`), on the FP64 matrix cores: the moved rows' basis values
// staged in the area 16 R at a time (padded by two: conflict-free operand
// reads), wave v the 16-column tiles v, v + 4, ... of Lambda, whose rows come
// from L2 once per chunk of rows.
__device__ void chain_rebuild(const SysDev& s, const WalkDev& w, int wk, int h, bool all, double* area, int area_bytes,
                              const double* r, int* list) {
  const int tid = chain_tid(), lane = tid & 63, wave = tid >> 6;
  const int n = h == 0 ? s.nu : s.nd, i0 = h == 0 ? 0 : s.nu, Lp = s.Lp, ldp = Lp + 2;
  const double* phi = (const double*)w.phi + ((long)wk * s.N + i0) * Lp;
  double* P = (double*)w.P + ((long)wk * s.N + i0) * Lp;
  double* rP = w.rpos_P + ((long)wk * s.N + i0) * 3;
  const double* lam = h == 0 ? s.lam : s.lamT;
  __syncthreads();   // the area's readers are done; basis rows are stored
  if (wave == 0) {
    const double* q = r + 3 * (i0 + lane);
    bool mv = false;
    if (lane < n) {
      mv = all || !(q[0] == rP[3 * lane] && q[1] == rP[3 * lane + 1] && q[2] == rP[3 * lane + 2]);
      if (mv) { rP[3 * lane] = q[0]; rP[3 * lane + 1] = q[1]; rP[3 * lane + 2] = q[2]; }
    }
    const unsigned long long b = __ballot(mv);
    if (mv) list[1 + __popcll(b & ((1ull << lane) - 1ull))] = lane;
    if (lane == 0) list[0] = __popcll(b);
  }
  __syncthreads();
  const int cnt = list[0];
  const int chunk = min(4, area_bytes / (8 * 16 * ldp)) * 16;
  for (int c0 = 0; c0 < cnt; c0 += chunk) {
    const int m = min(chunk, cnt - c0), RT = (m + 15) / 16;
    for (int q = tid; q < 16 * RT * (Lp / 2); q += kChainT) {
      const int i = q / (Lp / 2), k = 2 * (q - i * (Lp / 2));
      const double2 v = i < m ? *reinterpret_cast<const double2*>(phi + (long)list[1 + c0 + i] * Lp + k) : double2{0.0, 0.0};
      area[i * ldp + k] = v.x;
      area[i * ldp + k + 1] = v.y;
    }
    __syncthreads();
    const int li = lane & 15, lk = lane >> 4;
    for (int ct = wave; ct < Lp / 16; ct += 4) {
      const double* lc = lam + (long)lk * Lp + ct * 16 + li;
      cdx4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = cdx4{0.0, 0.0, 0.0, 0.0};
      double b[4], bn[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) b[u] = lc[(long)(4 * u) * Lp];
      for (int k = 0; k < Lp; k += 16) {
        const bool more = k + 16 < Lp;
#pragma unroll
        for (int u = 0; u < 4; ++u) bn[u] = more ? lc[(long)(k + 16 + 4 * u) * Lp] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double* a = area + li * ldp + k + 4 * u + lk;
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (t < RT) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[16 * t * ldp], b[u], acc[t], 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = bn[u];
      }
      // lane holds column lane % 16 and rows 4 r + lane / 16
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = 16 * t + 4 * q + lk;
          if (i < m) P[(long)list[1 + c0 + i] * Lp + ct * 16 + li] = acc[t][q];
        }
    }
    __syncthreads();
  }
}

enum { kRun = 0, kPropose = 1 };

// CON: the orbitals are contractions of Lq primitives; T: threads (512: large form only)
template <int MODE, bool SMALL, int QL, bool CON = false, int T = kChainT>
__global__ void __launch_bounds__(T, MODE == kRun ? 2 : 4) chain_kernel(SysDev s, WalkDev w, ChainArgs a) {
  constexpr int NW = T / 64;
  static_assert(!SMALL || T == kChainT, "the small form's LDS is for four waves");
  static_assert(MODE == kRun || !SMALL, "single moves of small systems take the per-move kernels");
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wk = blockIdx.x;
  const int n = s.nu, ld = chain_ld(n), N = s.N, L = s.L, Lp = s.Lp, np = s.ptn, LJ = s.LJ, nn = s.n_nuc;
  const long Wk = w.Wk;
  auto at = [&](int off) { return (double*)(lds + off); };
  double *area = at(a.ly.area), *B = at(a.ly.B), *r = at(a.ly.r), *nuc = at(a.ly.nuc), *draw = at(a.ly.draw),
         *red = at(a.ly.red), *part = at(a.ly.part), *ws = at(a.ly.ws), *cs = at(a.ly.cs), *lg = at(a.ly.lg);
  double* lv = at(a.ly.lv) + wave * a.cw;
  uint16_t* lm = (uint16_t*)(lds + a.ly.lm) + wave * a.cw;
  int *list = (int*)(lds + a.ly.list), *prow = (int*)(lds + a.ly.prow);
  double *Gv = at(a.ly.G), *jm = at(a.ly.jm), *chin = at(a.ly.chin), *jb = at(a.ly.jb);
  // chi, h and M: in LDS, or (large form) the walker's rows and the system's matrix
  double* chi = SMALL ? at(a.ly.chi) : w.chi + (long)wk * N * LJ;
  double* hv = SMALL ? at(a.ly.hv) : w.hv + (long)wk * N * LJ;
  const double* M3 = SMALL ? at(a.ly.M3) : s.M3;
  const int ldM = SMALL ? 2 * LJ + 1 : 2 * LJ;
  constexpr int JU = SMALL ? 1 : 8;   // loads of M in flight
  int* jk = (int*)(lds + a.ly.jk);
  double* Wg = w.W + (long)wk * n * n;
  double* phi = (double*)w.phi + (long)wk * N * Lp;
  // n x n passes: columns j, j + 1 of rows g, g + G, ... for thread (g, j / 2), g < G
  const int nh = (n + 1) / 2, G = a.groups, g = tid / nh, j = 2 * (tid - g * nh);
  // this thread's basis functions: 16 consecutive ones a wave in turn (what is
  // kept at r' lies close together), or every fourth one (all are kept)
  int mus[QL];
  double4 bf[QL];
  int bk[QL];
  double cm[QL];   // their column maxima (large form)
  int spin = a.e0 < n ? 0 : 1;   // (e0 < N)
#pragma unroll
  for (int q = 0; q < QL; ++q) {
    mus[q] = SMALL ? 4 * (64 * q + lane) + wave : T * q + ((lane >> 4) * NW + wave) * 16 + (lane & 15);
    const int mu = mus[q] < L ? mus[q] : 0;
    if (!CON) {
      bf[q] = s.bfn[mu];
      bk[q] = s.kind[mu];
    }
    cm[q] = SMALL ? 0.0 : w.cmax[((long)wk * 2 + 1 - spin) * Lp + mu];
  }
  double *qv = at(a.ly.qv), *cc = at(a.ly.cc);
  uint16_t* ci = (uint16_t*)(lds + a.ly.ci);
  int* cp = (int*)(lds + a.ly.cp);
  if (CON && a.con_lds) {
    for (int q = tid; q < s.nnz_con; q += T) {
      cc[q] = s.con_coef[q];
      ci[q] = (uint16_t)s.con_idx[q];
    }
    for (int q = tid; q <= L; q += T) cp[q] = s.con_ptr[q];
  }
  double* j2p = red + 2 * NW;
  if (tid < 8) j2p[tid] = s.j2d[tid];
  // state to LDS
  if (MODE == kRun)
    for (int q = tid; q < n * n; q += T) {
      const int i = q / n, k = q - i * n;
      B[spin == 0 ? i * ld + k : k * ld + i] = a.Ainv[(long)wk * n * n + q];
    }
  if (MODE == kRun && (n & 1))   // the column that makes the pairs
    for (int q = tid; q < n; q += T) B[q * ld + n] = 0.0;
  for (int q = tid; q < 3 * N; q += T) r[q] = w.r[(long)wk * 3 * N + q];
  for (int q = tid; a.nuc_lds && q < nn; q += T) {
    nuc[5 * q] = s.R[3 * q]; nuc[5 * q + 1] = s.R[3 * q + 1]; nuc[5 * q + 2] = s.R[3 * q + 2];
    nuc[5 * q + 3] = s.Z[q];
    nuc[5 * q + 4] = s.j1_b[q];
  }
  if constexpr (SMALL)
    for (int q = tid; q < N * LJ; q += T) {
      chi[q] = w.chi[(long)wk * N * LJ + q];
      hv[q] = w.hv[(long)wk * N * LJ + q];
    }
  for (int q = tid; q < 2 * LJ; q += T) {
    Gv[q] = w.G3[(long)wk * 2 * LJ + q];
    jm[q] = s.jm[q];
  }
  for (int q = tid; q < LJ; q += T) {
    const double4 f = s.jbfn[q];
    jb[4 * q] = f.x; jb[4 * q + 1] = f.y; jb[4 * q + 2] = f.z; jb[4 * q + 3] = f.w;
    jk[q] = s.jkind[q];
  }
  if constexpr (SMALL)
    for (int q = tid; q < 4 * LJ * LJ; q += T) at(a.ly.M3)[q / (2 * LJ) * ldM + q % (2 * LJ)] = s.M3[q];
  double la = w.logabs[wk], sg = w.sign[wk], Jt = w.J[wk];   // kept by thread 0
  int acc_n = 0, logs = 0;   // accepted moves; those whose ratio and Jastrow change wait in lg
  // log|Psi| of the waiting moves: their logarithms side by side in wave 0, the
  // sums in order (a logarithm a move in one lane would hold up every wave)
  auto fold_logs = [&]() {
    if (wave == 0) {
      double l = 0.0;
      if (lane < logs) l = log(fabs(lg[lane]));
      if (lane < logs) lg[lane] = l;
      __builtin_amdgcn_wave_barrier();
      if (lane == 0)
        for (int k = 0; k < logs; ++k) la += lg[k] + lg[kChainLogs + k];
    }
    logs = 0;
  };
  int since = a.since0, buf = a.buf_spin0, valid = a.valid0, half = -1;
  bool due = false;   // the last move filled the buffer: refresh
  // thread ranges of the Jastrow sums: the new and the old position and the
  // Jastrow basis start a wave apart, after the basis functions of the last pass
  const int nj = nn + N;
  const int off1 = (L + 63) / 64 * 64, off2 = off1 + (nj + 63) / 64 * 64, off3 = off2 + (nj + 63) / 64 * 64;
  const int t1 = (tid - off1) & (T - 1), t2 = (tid - off2) & (T - 1), t3 = (tid - off3) & (T - 1);
  const int lpf = 1 << a.lsh, fpl = 64 >> a.lsh;   // lanes a column takes, columns a load
  const int fg = lane >> a.lsh, rp = 2 * (lane & (lpf - 1));
  const bool row_ok = rp < np;

  auto jsum = [&](int t, int e, double px, double py, double pz) {
    double v = 0.0;
    for (int i = t; i < nj; i += T) {
      const bool isn = i < nn;
      const int je = i - nn;
      double x, y, z, Z = 0.0, b = 0.0;
      if (!isn) { x = r[3 * je]; y = r[3 * je + 1]; z = r[3 * je + 2]; }
      else if (a.nuc_lds) { const double* c = nuc + 5 * i; x = c[0]; y = c[1]; z = c[2]; Z = c[3]; b = c[4]; }
      else { x = s.R[3 * i]; y = s.R[3 * i + 1]; z = s.R[3 * i + 2]; Z = s.Z[i]; b = s.j1_b[i]; }
      const double dx = px - x, dy = py - y, dz = pz - z;
      const double d = sqrt(dx * dx + dy * dy + dz * dz);
      double f, f1, f2;
      if (isn) {
        if (s.j1_form) { j1_radial(s.j1_form, Z, b, d, f, f1, f2); v += f; }
      } else if (s.j2_form && je != e) {
        j2_radial(s.j2_form, j2p, (e < n) == (je < n), d, f, f1, f2);
        v += f;
      }
    }
    return v;
  };

  int e = a.e0 - 1;
  for (int t = 0;; ++t) {
    const bool last = MODE == kRun && t == a.steps;   // only a refresh that is due
    e = e + 1 == N ? 0 : e + 1;
    const int sp = last ? buf : (e < n ? 0 : 1), ie = sp == 0 ? e : e - n;
    bool fence = t == 0;   // LDS written since the last barrier
    if constexpr (SMALL) {
      // the per-move path's schedule
      if (due || (since > 0 && sp != buf)) {
        __syncthreads();
        for (int q = chain_tid(); q < n * n; q += T) {
          const int i = q / n, k = q - i * n;
          B[i * ld + k] = Wg[q];
        }
        __syncthreads();
        double ldet = 0.0, sdet = 0.0;
        const bool sing = chain_invert(B, n, ld, sp == 1, part, cs, prow, ldet, sdet);
        fold_logs();
        if (tid == 0) {
          la = sing ? -__builtin_inf() : ldet + Jt;
          sg = sdet;
          w.logdet[wk] = ldet;
          w.detsign[wk] = sdet;
          w.singular[wk] = sing ? 1 : 0;
        }
        spin = sp;
        since = 0;
        due = false;
      }
      if (last) break;
      if (sp != spin) {   // nothing buffered: turn the inverse over
        __syncthreads();
        const int ct = chain_tid();
        double x[kChainSmallN * kChainSmallN / T];
#pragma unroll
        for (int q = 0; q < kChainSmallN * kChainSmallN / T; ++q) {
          const int y = ct + T * q, i = y / n, c = y - i * n;
          x[q] = y < n * n ? B[i * ld + c] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kChainSmallN * kChainSmallN / T; ++q) {
          const int y = ct + T * q, i = y / n, c = y - i * n;
          if (y < n * n) B[c * ld + i] = x[q];
        }
        fence = true;
      }
      spin = buf = sp;
      const int hs = 1 - sp;   // the half of P this spin's moves stream
      if (!((valid >> hs) & 1)) {
        chain_rebuild(s, w, wk, hs, a.all_rows != 0, area, a.area_bytes, r, list);
        valid |= 1 << hs;
        half = -1;
      }
      if (half != hs) {
        __syncthreads();
        const int nrow = hs == 0 ? s.nu : s.nd;
        const double* P = (const double*)w.P + ((long)wk * N + (hs == 0 ? 0 : n)) * Lp;
        for (int q = chain_tid(); q < np * (Lp / 2); q += T) {
          const int i = q / (Lp / 2), mu = 2 * (q - i * (Lp / 2));
          double2 v = double2{0.0, 0.0};   // (the row that makes ptn even)
          if (i < n) v = *reinterpret_cast<const double2*>((i < nrow ? P + (long)i * Lp : s.Uph + (long)(i - nrow) * Lp) + mu);
          area[mu * np + i] = v.x;
          area[(mu + 1) * np + i] = v.y;
        }
        half = hs;
        fence = true;
      }
    } else if (last) {
      break;
    }
    if (MODE == kRun && t % kChainDraws == 0) {
      __syncthreads();
      for (int q = chain_tid(); q < 4 * kChainDraws; q += T) {
        const int k = q >> 2, c = q & 3;
        if (t + k < a.steps)
          draw[q] = c < 3 ? a.disp[((long)(t + k) * Wk + wk) * 3 + c] : a.unif[(long)(t + k) * Wk + wk];
      }
      fence = true;
    }
    if (fence) __syncthreads();

    const double* dv = draw + 4 * (t % kChainDraws);
    const double ox = r[3 * e], oy = r[3 * e + 1], oz = r[3 * e + 2];
    double px, py, pz;
    if constexpr (MODE == kRun) { px = ox + dv[0]; py = oy + dv[1]; pz = oz + dv[2]; }
    else {
      const double* p = (a.r_new ? a.r_new : a.disp) + 3 * (long)wk;
      px = p[0]; py = p[1]; pz = p[2];
      if (!a.r_new) { px += ox; py += oy; pz += oz; }
    }
    // the Jastrow basis state of e, ahead of its use (LJ <= T)
    double jchi = 0.0, jhv = 0.0;
    if (t3 < LJ) { jchi = chi[e * LJ + t3]; jhv = hv[e * LJ + t3]; }
    // the inverse's column (lanes: rows lane and lane + 64)
    double c0 = 0.0, c1 = 0.0, w0 = 0.0, w1 = 0.0, R, dJ;
    double sv[QL];
    if constexpr (MODE == kPropose) {
      const double* A = a.Ainv + (long)wk * n * n;
      if (lane < n) c0 = sp == 0 ? A[(long)lane * n + ie] : A[(long)ie * n + lane];
      if (lane + 64 < n) c1 = sp == 0 ? A[(long)(lane + 64) * n + ie] : A[(long)ie * n + lane + 64];
    } else {
      if (lane < n) c0 = B[lane * ld + ie];
      if (lane + 64 < n) c1 = B[(lane + 64) * ld + ie];
    }
    {
      // psi(r') of the wave's functions, the kept ones listed
      double thr = 0.0;
      if (!SMALL) {
        const double s1 = wave_sum(fabs(c0) + fabs(c1));
        thr = (s1 > 0.0) ? s.screen_tol() / ((double)L * s1) : 0.0;
      }
      int cnt = SMALL ? (L - wave + 3) / 4 : 0;
      if constexpr (CON) {   // (the last move's readers are past its sums)
        for (int mu = tid; mu < s.Lq; mu += T) qv[mu] = basis_value(s, mu, px, py, pz);
        __syncthreads();
      }
#pragma unroll
      for (int q = 0; q < QL; ++q) {
        sv[q] = 0.0;
        bool keep = false;
        if (mus[q] < L) {
          if constexpr (CON) {
            double v = 0.0;
            if (a.con_lds)
              for (int k = cp[mus[q]]; k < cp[mus[q] + 1]; ++k) v += cc[k] * qv[ci[k]];
            else
              for (int k = s.con_ptr[mus[q]]; k < s.con_ptr[mus[q] + 1]; ++k) v += s.con_coef[k] * qv[s.con_idx[k]];
            sv[q] = v;
          } else {
            sv[q] = basis_value_rec(bf[q], bk[q], px, py, pz);
          }
          keep = !(fabs(sv[q]) * cm[q] <= thr);
        }
        if constexpr (SMALL) {   // function k of the wave is 4 k + wave
          lv[64 * q + lane] = sv[q];
          continue;
        }
        const unsigned long long b = __ballot(keep);
        if (keep) {
          const int k = cnt + __popcll(b & ((1ull << lane) - 1ull));
          lm[k] = (uint16_t)mus[q];
          lv[k] = sv[q];
        }
        cnt += __popcll(b);
      }
      __builtin_amdgcn_wave_barrier();   // (the list is the wave's own: its LDS accesses run in order)
      // their columns: the wave's share of the new row (column) of W
      // (32-bit offsets: a walker's transposed rows are at most 2 MB)
      const char* src = SMALL ? (const char*)area : (const char*)(w.PT + (long)wk * Lp * s.pt_ld() + (sp == 0 ? np : 0));
      const uint32_t col = 8u * (uint32_t)(SMALL ? np : s.pt_ld());
      constexpr int U = SMALL ? 4 : (QL > 3 || MODE == kPropose ? kChainU - 2 : kChainU);
      double ax = 0.0, ay = 0.0;
      for (int k0 = fg; k0 - fg < cnt; k0 += U * fpl) {
        double2 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = k0 + u * fpl;
          x[u] = double2{0.0, 0.0};
          const uint32_t mu = SMALL ? 4u * (uint32_t)k + (uint32_t)wave : (uint32_t)lm[k < cnt ? k : 0];
          if (k < cnt && row_ok) x[u] = *reinterpret_cast<const double2*>(src + (mu * col + 8u * (uint32_t)rp));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = k0 + u * fpl;
          const double v = k < cnt ? lv[k] : 0.0;
          ax += v * x[u].x;
          ay += v * x[u].y;
        }
      }
      ax = lane_group_sum(ax, lpf);
      ay = lane_group_sum(ay, lpf);
      double* pt = part + (t & 1) * a.pst + wave * np;
      if (lane < lpf && row_ok) { pt[rp] = ax; pt[rp + 1] = ay; }
      // the Jastrow change
      double dj = jsum(t1, e, px, py, pz) - jsum(t2, e, ox, oy, oz);
      if (t3 < LJ) {
        const double4 f = double4{jb[4 * t3], jb[4 * t3 + 1], jb[4 * t3 + 2], jb[4 * t3 + 3]};
        const double v = basis_value_rec(f, jk[t3], px, py, pz);
        chin[t3] = v;
        dj += (v - jchi) * (Gv[sp * LJ + t3] - jhv + jm[sp * LJ + t3]);
      }
      dj = wave_sum(dj);
      if (lane == 0) red[NW * (t & 1) + wave] = dj;
      if (!SMALL && lane == 0) prow[wave] = cnt;   // (at the end: the last proposal's)
      __syncthreads();
      const double* ps = part + (t & 1) * a.pst;
      auto rows = [&]() {
        if (lane < n) {
          w0 = ps[lane];
#pragma unroll
          for (int q = 1; q < NW; ++q) w0 += ps[q * np + lane];
        }
        if (lane + 64 < n) {
          w1 = ps[lane + 64];
#pragma unroll
          for (int q = 1; q < NW; ++q) w1 += ps[q * np + lane + 64];
        }
      };
      rows();
      if constexpr (NW == 8) __syncthreads();   // (one buffer of partial sums)
      R = wave_sum(w0 * c0 + w1 * c1);
      if constexpr (!SMALL) {
        if (s.screen_again(R)) {   // uniform: the wave's functions left out that matter beside R
          const double lo = thr * s.screen_rest(R);
          int rest = 0;
          const int rt = chain_tid();   // (mus and cm anew: nothing more is held in registers up to here)
#pragma unroll
          for (int q = 0; q < QL; ++q) {
            const int mu = T * q + (((rt & 63) >> 4) * NW + (rt >> 6)) * 16 + (rt & 15);
            const double v = mu < L ? fabs(sv[q]) * w.cmax[((long)wk * 2 + 1 - sp) * Lp + mu] : 0.0;
            const bool more = v > lo && v <= thr;
            const unsigned long long b = __ballot(more);
            if (more) {
              const int k = rest + __popcll(b & ((1ull << lane) - 1ull));
              lm[k] = (uint16_t)mu;
              lv[k] = sv[q];
            }
            rest += __popcll(b);
          }
          __builtin_amdgcn_wave_barrier();
          double bx = 0.0, by = 0.0;
#pragma unroll 4
          for (int k = fg; k < rest; k += fpl)
            if (row_ok) {
              const double2 x = *reinterpret_cast<const double2*>(src + ((uint32_t)lm[k] * col + 8u * (uint32_t)rp));
              bx += lv[k] * x.x;
              by += lv[k] * x.y;
            }
          bx = lane_group_sum(bx, lpf);
          by = lane_group_sum(by, lpf);
          if constexpr (NW == 4) __syncthreads();   // the kept functions' sums are read
          if (lane < lpf && row_ok) { pt[rp] += bx; pt[rp + 1] += by; }
          __syncthreads();
          rows();
          if constexpr (NW == 8) __syncthreads();
          R = wave_sum(w0 * c0 + w1 * c1);
        }
      }
      const double* rd = red + NW * (t & 1);
      dJ = rd[0];
#pragma unroll
      for (int q = 1; q < NW; ++q) dJ += rd[q];
    }
    const double ratio = R * exp(dJ);
    if constexpr (MODE == kPropose) {
      // the pending proposal
      if (wave == 0) {
        if (lane < n) { w.w_new[(long)wk * n + lane] = w0; w.cvec[(long)wk * n + lane] = c0; }
        if (lane + 64 < n) { w.w_new[(long)wk * n + lane + 64] = w1; w.cvec[(long)wk * n + lane + 64] = c1; }
      }
#pragma unroll
      for (int q = 0; q < QL; ++q)
        if (mus[q] < L) w.psi_new[(long)wk * Lp + mus[q]] = sv[q];
      for (int k = tid; k < LJ; k += T) w.chi_new[(long)wk * LJ + k] = chin[k];
      if (tid == 0) {
        w.r_new[3 * wk] = px; w.r_new[3 * wk + 1] = py; w.r_new[3 * wk + 2] = pz;
        w.rdet[wk] = R;
        w.ratio[wk] = ratio;
        w.dJ[wk] = dJ;
        {
          int kept = 0;
          for (int q = 0; q < NW; ++q) kept += prow[q];
          w.nkeep[wk] = kept;
        }
        if (a.ratio_out) a.ratio_out[wk] = ratio;
      }
      return;
    }
    const bool acc = dv[3] < ratio * ratio;   // uniform
    if (acc) {
      // every wave writes the same w and column: its own reads need no barrier
      if (lane < n) { ws[lane] = w0; cs[lane] = c0; }
      if (lane + 64 < n) { ws[lane + 64] = w1; cs[lane + 64] = c1; }
      __builtin_amdgcn_wave_barrier();
      const double ir = 1.0 / R;
      double* pu = part + ((t + 1) & 1) * a.pst;   // (the previous move's partial sums are read)
      if (g < G) {
        double2 u = double2{0.0, 0.0};
#pragma unroll 4
        for (int i = g; i < n; i += G) {
          const double2 b = *reinterpret_cast<const double2*>(B + i * ld + j);
          u.x = fma(ws[i], b.x, u.x);
          u.y = fma(ws[i], b.y, u.y);
        }
        pu[2 * (g * nh) + j] = u.x;
        pu[2 * (g * nh) + j + 1] = u.y;
      }
      if (wave == 0) {
        if (lane < n) Wg[sp == 0 ? (long)ie * n + lane : (long)lane * n + ie] = w0;
        if (lane + 64 < n) Wg[sp == 0 ? (long)ie * n + lane + 64 : (long)(lane + 64) * n + ie] = w1;
      }
#pragma unroll
      for (int q = 0; q < QL; ++q)
        if (mus[q] < L) phi[(long)e * Lp + mus[q]] = sv[q];
      // [G_u; G_d] += M3[:, s] (chi(r') - chi_e), h_e = M^{ss} chi(r'): four lanes a sum
      for (int q = tid; q < 12 * LJ; q += T) {
        const int o = q >> 2, sub = q & 3;
        const bool first = o < 2 * LJ;
        const double* row = M3 + (first ? o : sp * LJ + o - 2 * LJ) * ldM + sp * LJ;
        double v = 0.0;
#pragma unroll JU
        for (int k = sub; k < LJ; k += 4) v += row[k] * (first ? chin[k] - chi[e * LJ + k] : chin[k]);
        v += dpp_f64<0xB1>(v);
        v += dpp_f64<0x4E>(v);
        if (sub == 0) {
          if (first) Gv[o] += v;
          else hv[e * LJ + o - 2 * LJ] = v;
        }
      }
      __syncthreads();
      if (g < G) {
        double2 u = *reinterpret_cast<const double2*>(pu + j);
        for (int q = 1; q < G; ++q) {
          const double2 v = *reinterpret_cast<const double2*>(pu + 2 * q * nh + j);
          u.x += v.x;
          u.y += v.y;
        }
        if (j == ie) u.x -= 1.0;
        if (j + 1 == ie) u.y -= 1.0;
        u.x *= ir;
        u.y *= ir;
#pragma unroll 4
        for (int i = g; i < n; i += G) {
          double2* p = reinterpret_cast<double2*>(B + i * ld + j);
          const double2 b = *p;
          const double ci = cs[i];
          *p = double2{fma(-ci, u.x, b.x), fma(-ci, u.y, b.y)};
        }
      }
      for (int k = tid; k < LJ; k += T) chi[e * LJ + k] = chin[k];
      if (tid == 0) {
        r[3 * e] = px; r[3 * e + 1] = py; r[3 * e + 2] = pz;
        if (R < 0.0) sg = -sg;
        Jt += dJ;
        lg[logs] = R;
        lg[kChainLogs + logs] = dJ;
      }
      acc_n += 1;
      logs += 1;
      if (MODE == kRun && logs == kChainLogs) fold_logs();
      __syncthreads();
    }
    valid &= ~(1 << sp);
    since += 1;
    due = SMALL && since >= a.cap;
  }

  // the walker's state back
  if (MODE == kRun) fold_logs();
  __syncthreads();
  if (SMALL || a.store_A)
    for (int q = tid; q < n * n; q += T) {
      const int i = q / n, k = q - i * n;
      w.A[(long)wk * n * n + q] = B[spin == 0 ? i * ld + k : k * ld + i];
    }
  for (int q = tid; q < 3 * N; q += T) w.r[(long)wk * 3 * N + q] = r[q];
  if constexpr (SMALL)
    for (int q = tid; q < N * LJ; q += T) {
      w.chi[(long)wk * N * LJ + q] = chi[q];
      w.hv[(long)wk * N * LJ + q] = hv[q];
    }
  for (int q = tid; q < 2 * LJ; q += T) w.G3[(long)wk * 2 * LJ + q] = Gv[q];
  if (tid == 0) {
    w.logabs[wk] = la;
    w.sign[wk] = sg;
    w.J[wk] = Jt;
    if (SMALL) w.wm[wk] = 0;
    // the functions the last proposal read
    if (MODE == kRun) {
      int kept = SMALL ? L : 0;
      for (int q = 0; !SMALL && q < NW; ++q) kept += prow[q];
      w.nkeep[wk] = kept;
    }
    if (MODE == kRun && a.cnt) a.cnt[wk] += acc_n;
  }
}

// ---------------------------------------------------------------------------
// The accept of a single pending proposal of electron e (large form): the run's
// update of the inverse, kAccCols of its columns (rows for a down move: B is the
// transpose) a workgroup.  A column's sum over w and its update need that column
// alone, beside w and column e, which the proposal left in cvec; thread (g, k) holds
// the entries g, g + G, ... of column k in registers from the sum to the update, in
// the run's order of sums (bitwise the run's).  The first workgroup also takes the
// W line, the basis row, the Jastrow state and the sums.  Decided by acc (the
// caller's) or by unif.
// Bound by HBM: 16 n^2 bytes an accepted walker.  us for a proposal and its accept of 60 %
// of 1024 walkers, all of the inverse staged in LDS by one workgroup (131 KB at n = 127, one
// a compute unit) -> here: n = 127 226 -> 114 (refined 205 -> 105), n = 96 135 -> 63, n = 80
// 67 -> 46; 16 walkers, n = 127 42 -> 28.  The delayed form of the per-move kernels, which
// moves 3 m n numbers for m buffered moves, is still ahead of it past n = 112 at 1024
// walkers (refined, n = 127: 96).
// Transposed tiles (down moves) go through LDS, both ways in whole lines.
// ---------------------------------------------------------------------------
constexpr int kAccCols = 32, kAccLd = kAccCols + 1;

template <int RP>   // entries a thread: ceil(n / G)
__global__ void __launch_bounds__(kAccCols * kChainG) chain_accept_kernel(SysDev s, WalkDev w, int e, int G, int tiles,
                                                                          const uint8_t* __restrict__ acc_in,
                                                                          const double* __restrict__ unif,
                                                                          int32_t* __restrict__ cnt) {
  extern __shared__ __align__(16) char lds[];   // down: the tile, [n][kAccLd]
  __shared__ double ws[kChainMaxN], cs[kChainMaxN], part[kChainG][kAccCols];
  const int wk = blockIdx.x / tiles, tile = blockIdx.x - wk * tiles, T = blockDim.x;
  const int tid = threadIdx.x, n = s.nu, sp = e < n ? 0 : 1, ie = sp == 0 ? e : e - n;
  const double R = w.rdet[wk], ratio = w.ratio[wk];
  const bool acc = unif ? unif[wk] < ratio * ratio : acc_in[wk] != 0;
  if (tile == 0 && tid == 0) w.acc[wk] = acc ? 1 : 0;
  if (!acc) return;   // uniform
  double* A = w.A + (long)wk * n * n;
  double* tl = (double*)lds;
  const int k0 = tile * kAccCols, nc = min(kAccCols, n - k0);
  const int g = tid / kAccCols, c = tid - g * kAccCols;
  const bool ok = g < G && c < nc;
  double b[RP];
  if (sp == 0) {
#pragma unroll
    for (int q = 0; q < RP; ++q) {
      const int i = g + G * q;
      b[q] = ok && i < n ? A[(long)i * n + k0 + c] : 0.0;
    }
  } else {   // (nc n <= RP T entries, rows of A side by side)
#pragma unroll
    for (int q = 0; q < RP; ++q) b[q] = tid + T * q < nc * n ? A[(long)k0 * n + tid + T * q] : 0.0;
  }
  double* Wg = w.W + (long)wk * n * n;
  for (int j = tid; j < n; j += T) {
    const double x = w.w_new[(long)wk * n + j];
    ws[j] = x;
    cs[j] = w.cvec[(long)wk * n + j];
    if (tile == 0) Wg[sp == 0 ? (long)ie * n + j : (long)j * n + ie] = x;
  }
  if (tile == 0) {   // (their round trips under the tile's)
    double* phi = (double*)w.phi + ((long)wk * s.N + e) * s.Lp;
#pragma unroll 4
    for (int mu = tid; mu < s.L; mu += T) phi[mu] = w.psi_new[(long)wk * s.Lp + mu];
    if (tid == 0) {
      const double dJ = w.dJ[wk];
      for (int k = 0; k < 3; ++k) w.r[((long)wk * s.N + e) * 3 + k] = w.r_new[3 * (long)wk + k];
      w.logabs[wk] += log(fabs(R)) + dJ;
      if (R < 0.0) w.sign[wk] = -w.sign[wk];
      w.J[wk] += dJ;
      if (cnt) cnt[wk] += 1;
    }
  }
  // entry x of the tile: row i, column k (x < 2^12 and 1 / n to 24 bits: exact)
  const float rn = 1.0f / (float)n;
  auto at = [&](int x) {
    const int k = (int)(((float)x + 0.5f) * rn), i = x - k * n;
    return i * kAccLd + k;
  };
  if (sp == 1) {
#pragma unroll
    for (int q = 0; q < RP; ++q)
      if (tid + T * q < nc * n) tl[at(tid + T * q)] = b[q];
  }
  __syncthreads();
  if (sp == 1) {
#pragma unroll
    for (int q = 0; q < RP; ++q) {
      const int i = g + G * q;
      b[q] = ok && i < n ? tl[i * kAccLd + c] : 0.0;
    }
  }
  double u = 0.0;
#pragma unroll
  for (int q = 0; q < RP; ++q)
    if (g + G * q < n && ok) u = fma(ws[g + G * q], b[q], u);
  if (g < G) part[g][c] = u;
  __syncthreads();
  if (ok) {
    u = part[0][c];
    for (int q = 1; q < G; ++q) u += part[q][c];
    if (k0 + c == ie) u -= 1.0;
    u *= 1.0 / R;
#pragma unroll
    for (int q = 0; q < RP; ++q) {
      const int i = g + G * q;
      if (i < n) {
        const double v = fma(-cs[i], u, b[q]);
        if (sp == 0) A[(long)i * n + k0 + c] = v;
        else tl[i * kAccLd + c] = v;
      }
    }
  }
  if (sp == 1) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RP; ++q)
      if (tid + T * q < nc * n) A[(long)k0 * n + tid + T * q] = tl[at(tid + T * q)];
  }
  if (tile || !s.LJ) return;
  // the run's update of the Jastrow basis state
  const int LJ = s.LJ;
  const double* chin = w.chi_new + (long)wk * LJ;
  double *ce = w.chi + ((long)wk * s.N + e) * LJ, *he = w.hv + ((long)wk * s.N + e) * LJ, *Gv = w.G3 + (long)wk * 2 * LJ;
  for (int q = tid; q < 12 * LJ; q += T) {
    const int o = q >> 2, sub = q & 3;
    const bool first = o < 2 * LJ;
    const double* row = s.M3 + (long)(first ? o : sp * LJ + o - 2 * LJ) * 2 * LJ + sp * LJ;
    double v = 0.0;
#pragma unroll 8
    for (int k = sub; k < LJ; k += 4) v += row[k] * (first ? chin[k] - ce[k] : chin[k]);
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    if (sub == 0) {
      if (first) Gv[o] += v;
      else he[o - 2 * LJ] = v;
    }
  }
  __syncthreads();   // chi_e is read
  for (int k = tid; k < LJ; k += T) ce[k] = chin[k];
}

// Threads of a large form: past 80 KiB one workgroup has a compute unit to itself, and
// with four waves each SIMD waits on one wave's LDS and cache round trips.  Eight waves
// of the same LDS (one buffer of partial sums and a barrier more a move in place of two
// buffers); us a move of a sweep, 256 / 512 threads: n = 96 FP64 16 walkers 13.5/11.3,
// 256 17.0/14.2, 1024 63.5/53.2, QMC_REFINED 1024 61.3/52.8; n = 128 FP64 256 walkers
// 26.3/23.4, QMC_REFINED 1024 83.1/73.4.  (n = 80, two workgroups a compute unit: 256.)
static int chain_threads(const SysDev& s) {
  ChainArgs a{};
  return chain_layout(s, false, a).total <= kChainMaxLds / 2 ? kChainT : 2 * kChainT;
}

// The form that takes a system: FP64 rows and a walker's state within the LDS (0:
// neither).
int chain_class(const SysDev& s, const WalkDev& w) {
  if (!s.screened() || s.nu > kChainMaxN || s.L > 1024 || !w.rpos_P || !w.PT || s.Lp % 32) return 0;
  if (s.LJ > kChainT || s.N > 4096 || s.n_nuc > 4096) return 0;
  ChainArgs a{};
  if (s.nu <= kChainSmallN && s.L <= 2 * kChainT && chain_layout(s, true, a).total <= kChainSmallLds) return 1;
  return chain_layout(s, false, a, false, chain_threads(s)).total <= kChainMaxLds ? 2 : 0;
}

// A run stages the inverse in LDS and stores it again, 16 n^2 bytes a walker, for as
// many walkers at a time as the LDS lets the chip hold: with r such rounds a run of up to
// r moves (r - 1 with 512 threads) is cheaper as single proposals and accepts, which touch
// the inverse of accepting walkers alone and fill the chip whatever their LDS.  us a move,
// run / single, for runs of 1, 2, 3, 4, 8: n = 80, 256 walkers (r = 1) 27/23 19/23 15/23 14/22
// 10/21; n = 80, 1024 (2) 60/36 39/34 32/32 28/32 23/31; n = 40, 2048 (4) 57/33 38/31 31/29 29/29
// 24/28; n = 96, 512 (2) 56/40 42/41 37/41 34/41 30/41; n = 96, 1024 (4) 110/73 85/74 77/75 72/75
// 63/75; n = 127, 256 (1) 48/44 37/45 33/45 31/45 28/46; n = 127, 1024 (4) 178/125 138/129 120/131
// 110/132 94/133.
int chain_single(const SysDev& s, const WalkDev& w) {
  const bool two = chain_threads(s) == kChainT;   // workgroups a compute unit
  const int at_once = two ? 512 : 256, rounds = (w.Wk + at_once - 1) / at_once;
  return two ? rounds : std::max(1, rounds - 1);
}

static hipError_t chain_launch(const SysDev& s, const WalkDev& w, int mode, ChainArgs& a, hipStream_t st,
                               hipEvent_t ev_start, hipEvent_t ev_stop) {
  const int cls = chain_class(s, w);
  if (cls == 0 || (mode != kRun && cls != 2) || a.steps < 1) return hipErrorInvalidValue;
  a.cap = wb_cap(s);
  const int T = cls == 1 ? kChainT : chain_threads(s);
  a.ly = chain_layout(s, cls == 1, a, mode == kPropose, T);
  const dim3 grid(w.Wk), blk(T);
#define QMC_CHAIN(M, S, Q) QMC_LAUNCH_EV((chain_kernel<M, S, Q>), grid, blk, a.ly.total, st, ev_start, ev_stop, s, w, a)
#define QMC_CHAIN_Q(M)                                                         \
  if (s.L <= kChainT) { QMC_CHAIN(M, false, 1); }                              \
  else if (s.L <= 2 * kChainT) { QMC_CHAIN(M, false, 2); }                     \
  else if (s.L <= 3 * kChainT) { QMC_CHAIN(M, false, 3); }                     \
  else { QMC_CHAIN(M, false, 4); }
  if (T == 2 * kChainT) {
#define QMC_CHAIN_2(M, Q, C) QMC_LAUNCH_EV((chain_kernel<M, false, Q, C, 2 * kChainT>), grid, blk, a.ly.total, st, ev_start, ev_stop, s, w, a)
#define QMC_CHAIN_2Q(M)                                                                               \
  if (s.Lq > 0) { QMC_CHAIN_2(M, 2, true); }                                                          \
  else if (s.L <= T) { QMC_CHAIN_2(M, 1, false); }                                                    \
  else { QMC_CHAIN_2(M, 2, false); }
    if (mode == kRun) { QMC_CHAIN_2Q(kRun) }
    else { QMC_CHAIN_2Q(kPropose) }
#undef QMC_CHAIN_2Q
#undef QMC_CHAIN_2
    return hipGetLastError();
  }
  if (s.Lq > 0) {
#define QMC_CHAIN_C(M, S, Q) QMC_LAUNCH_EV((chain_kernel<M, S, Q, true>), grid, blk, a.ly.total, st, ev_start, ev_stop, s, w, a)
    if (cls == 1) { QMC_CHAIN_C(kRun, true, 2); }
    else if (mode == kRun && s.L <= 2 * kChainT) { QMC_CHAIN_C(kRun, false, 2); }
    else if (mode == kRun) { QMC_CHAIN_C(kRun, false, 4); }
    else if (s.L <= 2 * kChainT) { QMC_CHAIN_C(kPropose, false, 2); }
    else { QMC_CHAIN_C(kPropose, false, 4); }
#undef QMC_CHAIN_C
    return hipGetLastError();
  }
  if (cls == 1) {
    if (s.L <= kChainT) { QMC_CHAIN(kRun, true, 1); }
    else { QMC_CHAIN(kRun, true, 2); }
  } else if (mode == kRun) { QMC_CHAIN_Q(kRun) }
  else { QMC_CHAIN_Q(kPropose) }
#undef QMC_CHAIN_Q
#undef QMC_CHAIN
  return hipGetLastError();
}

hipError_t launch_chain(const SysDev& s, const WalkDev& w, int e0, int steps, const double* disp, const double* unif,
                        int32_t* accept_count, int since0, int buf_spin0, int valid0, bool all_rows, bool store_A,
                        const double* Ainv, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  ChainArgs a{};
  a.e0 = e0 % s.N; a.steps = steps; a.since0 = since0; a.buf_spin0 = buf_spin0; a.valid0 = valid0;
  a.all_rows = all_rows ? 1 : 0; a.store_A = store_A ? 1 : 0;
  a.Ainv = Ainv; a.disp = disp; a.unif = unif; a.cnt = accept_count;
  return chain_launch(s, w, kRun, a, st, ev_start, ev_stop);
}

hipError_t launch_chain_propose(const SysDev& s, const WalkDev& w, int e, const double* r_new, const double* disp,
                                double* ratio, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  ChainArgs a{};
  a.e0 = e; a.steps = 1; a.Ainv = w.A; a.r_new = r_new; a.disp = disp; a.ratio_out = ratio;
  return chain_launch(s, w, kPropose, a, st, ev_start, ev_stop);
}

hipError_t launch_chain_accept(const SysDev& s, const WalkDev& w, int e, const uint8_t* acc, const double* unif,
                               int32_t* accept_count, hipStream_t st) {
  if (chain_class(s, w) != 2 || s.nu > kChainMaxN || (!acc && !unif)) return hipErrorInvalidValue;
  const int n = s.nu, G = chain_groups(n, chain_threads(s)), tiles = (n + kAccCols - 1) / kAccCols;
  const long total = (long)tiles * w.Wk;
  if (total > 0x7fffffffL) return hipErrorInvalidValue;
  const size_t lds = e < n ? 0 : sizeof(double) * (size_t)n * kAccLd;
  const dim3 grid((unsigned)total), blk(kAccCols * ((G + 1) / 2 * 2));
#define QMC_ACC(RP) hipLaunchKernelGGL(chain_accept_kernel<RP>, grid, blk, lds, st, s, w, e, G, tiles, acc, unif, accept_count)
  const int rp = (n + G - 1) / G;
  if (rp <= 8) QMC_ACC(8);
  else if (rp <= 16) QMC_ACC(16);
  else QMC_ACC(32);   // (n <= 128: G >= 4)
#undef QMC_ACC
  return hipGetLastError();
}

}  // namespace qmc
