// Resident chain: a whole run of Metropolis moves of a small system in one
// launch, one workgroup per walker, refreshes, changes of spin and P rebuilds
// included.
//
// What bounds small systems is latency: with a launch per phase a move of 20
// electrons is some thirty dependent trips to memory (25.7 us a move at 256
// walkers x 20 e, L = 44 with a Jastrow basis, 2.1 ms of a 2.9 ms run of 100
// moves; the arithmetic of a move is well under 1 us).  Nothing in a move
// leaves its walker, so one workgroup keeps the walker's state in LDS and the
// moves follow each other with two barriers for a rejected move and four for
// an accepted one:
//   draws (64 steps at a time), positions, nuclei, the Jastrow basis state;
//   the streamed half of P transposed, PT[mu][j] (all of it is read: at these
//   sizes the screening would cost more than the skipped columns);
//   the inverse itself in the orientation of the moving spin, B = W^{-1} for up
//   moves, its transpose for down moves, so that both spins read column e and
//   update by the same Sherman-Morrison step
//     R = sum_j w_j B[j][e],  B[j][k] -= B[j][e] (sum_i w_i B[i][k] - delta_ek) / R.
// W's row or column, the basis row and (at a rebuild) the P rows go to the
// walker's arrays in global memory, which hold the usual state at the end with
// an empty delayed-update buffer.  The refresh and rebuild schedule is that of
// the per-move path.
#include <hip/hip_ext.h>

#include "internal.h"
#include <algorithm>

namespace qmc {

constexpr int kChainT = 256;        // threads
constexpr int kChainMaxN = 64;      // rows of W (one per lane)
constexpr int kChainDraws = 64;     // steps whose draws are staged together
constexpr int kChainMaxLds = 80 * 1024;   // two workgroups per compute unit

struct ChainLayout {   // byte offsets in LDS
  int area, B, psi, r, nuc, draw, red, part, pu, list, prow, chi, hv, G, jm, chin, jb, jk, M3, total;
};

struct ChainArgs {
  int e0, steps;            // first electron, moves
  int cap;                  // attempts of one spin between refreshes
  int since0, buf_spin0;    // schedule state at the start
  int valid0;               // P halves that hold (bit 0 up, 1 down)
  int all_rows;             // rebuild every row of a half, not only the moved ones
  const double* Ainv;       // [Wk][n][n] the inverse at the start
  const double* disp;       // [steps][Wk][3]
  const double* unif;       // [steps][Wk]
  int32_t* cnt;             // [Wk] or null
  int area_bytes;
  ChainLayout ly;
};

static ChainLayout chain_layout(const SysDev& s, int& area_bytes) {
  ChainLayout o{};
  const int n = s.nu, ld = n | 1, f8 = 8;
  area_bytes = f8 * std::max(s.ptn * s.Lp, 16 * (s.Lp + 2));
  int at = 0;
  auto take = [&](int& p, int bytes) { p = at; at += (bytes + 15) / 16 * 16; };
  take(o.area, area_bytes);
  take(o.B, f8 * n * ld);
  take(o.psi, f8 * s.Lp);
  take(o.r, f8 * 3 * s.N);
  take(o.nuc, f8 * 5 * s.n_nuc);
  take(o.draw, f8 * 4 * kChainDraws);
  take(o.red, f8 * 16);   // partial sums of two moves, the two-body parameters
  take(o.part, f8 * 4 * kChainMaxN);
  take(o.pu, f8 * 4 * kChainMaxN);
  take(o.list, 4 * (kChainMaxN + 1));
  take(o.prow, 4 * kChainMaxN);
  if (s.LJ > 0) {
    take(o.chi, f8 * s.N * s.LJ);
    take(o.hv, f8 * s.N * s.LJ);
    take(o.G, f8 * 2 * s.LJ);
    take(o.jm, f8 * 2 * s.LJ);
    take(o.chin, f8 * s.LJ);
    take(o.jb, f8 * 4 * s.LJ);
    take(o.jk, 4 * s.LJ);
    take(o.M3, f8 * 2 * s.LJ * (2 * s.LJ + 1));
  }
  o.total = at;
  return o;
}

// B[n][ld] (LDS) <- its inverse, in place: Gauss-Jordan with the pivot of step k
// the largest |entry| of column k among the rows not yet pivoted (lowest row on
// ties; the row kernel's choice).  KP: columns per thread row, a power of two
// >= n.  Afterwards element (p_k, k') holds inverse element (k, p_k'), which the
// last step puts in place, transposed when tr.  log|det| and sign to every
// thread of wave 0; singular: returns true and B is not a number.
template <int KP>
__device__ bool chain_invert(double* B, int n, int ld, bool tr, int* prow, double& logdet, double& sign) {
  constexpr int G = kChainT / KP, NQ = (KP + G - 1) / G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int j = tid & (KP - 1), g = tid / KP;
  bool used = lane >= n;
  double own = 1.0;
  int own_p = lane;
  for (int k = 0; k < n; ++k) {
    const double f = lane < n ? B[lane * ld + k] : 0.0;
    const unsigned long long key =
        used ? 0ull : ((__double_as_longlong(fabs(f)) & ~0xFFull) | (unsigned long long)(255 - lane));
    const unsigned long long best = wave_max_u64(key);
    const int p = 255 - (int)(best & 0xFFull);
    const double piv = best ? __shfl(f, p & 63, 64) : 0.0;
    if (!(piv != 0.0)) {   // the same for every wave
      __syncthreads();
      const double nanv = __longlong_as_double(0x7ff8000000000000LL);
      for (int q = tid; q < n * ld; q += kChainT) B[q] = nanv;
      __syncthreads();
      logdet = -__builtin_inf();
      sign = 0.0;
      return true;
    }
    if (lane == p) used = true;
    if (lane == k) { own = piv; own_p = p; }
    const double ip = 1.0 / piv;
    double t[NQ], fi[NQ];
    const double pr = j < n ? B[p * ld + j] : 0.0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int i = g + G * q;
      const bool ok = i < n && j < n;
      fi[q] = ok ? B[i * ld + k] : 0.0;
      t[q] = ok ? B[i * ld + j] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int i = g + G * q;
      if (i < n && j < n) {
        const double gi = fi[q] * ip;
        double v;
        if (i == p) v = j == k ? ip : pr * ip;
        else v = j == k ? -gi : fma(-gi, pr, t[q]);
        B[i * ld + j] = v;
      }
    }
    __syncthreads();
  }
  if (tid < n) prow[tid] = own_p;   // wave 0's lanes
  double t[NQ];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = g + G * q;
    t[q] = i < n && j < n ? B[prow[i] * ld + j] : 0.0;   // inverse element (i, prow[j])
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = g + G * q;
    if (i < n && j < n) B[tr ? prow[j] * ld + i : i * ld + prow[j]] = t[q];
  }
  if (tid < 64) {
    int odd = 0;
    if (lane < n) {
      odd = own < 0.0;
      for (int k2 = lane + 1; k2 < n; ++k2) odd += prow[k2] < own_p;
    }
    const double ls = wave_sum(lane < n ? log(fabs(own)) : 0.0);
    for (int o = 32; o > 0; o >>= 1) odd += __shfl_xor(odd, o, 64);
    logdet = ls;
    sign = (odd & 1) ? -1.0 : 1.0;
  }
  __syncthreads();
  return false;
}

typedef double cdx4 __attribute__((ext_vector_type(4)));

// The P rows of half h whose electron has moved since they were built (all of
// them with `all`), on the FP64 matrix cores: the moved rows' basis values
// staged in the area 16 R at a time (padded by two: conflict-free operand
// reads), wave v the 16-column tiles v, v + 4, ... of Lambda, whose rows come
// from L2 once per chunk of rows.
__device__ void chain_rebuild(const SysDev& s, const WalkDev& w, int wk, int h, bool all, double* area, int area_bytes,
                              const double* r, int* list) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
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

template <int KP, int QL>
__global__ void __launch_bounds__(kChainT, 2) chain_kernel(SysDev s, WalkDev w, ChainArgs a) {
  extern __shared__ __align__(16) char lds[];
  constexpr int G = kChainT / KP, NQ = (KP + G - 1) / G;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wk = blockIdx.x;
  const int n = s.nu, ld = n | 1, N = s.N, L = s.L, Lp = s.Lp, np = s.ptn, LJ = s.LJ, nn = s.n_nuc;
  const long Wk = w.Wk;
  auto at = [&](int off) { return (double*)(lds + off); };
  double *area = at(a.ly.area), *B = at(a.ly.B), *psi = at(a.ly.psi), *r = at(a.ly.r), *nuc = at(a.ly.nuc),
         *draw = at(a.ly.draw), *red = at(a.ly.red), *part = at(a.ly.part), *pu = at(a.ly.pu);
  int *list = (int*)(lds + a.ly.list), *prow = (int*)(lds + a.ly.prow);
  double *chi = at(a.ly.chi), *hv = at(a.ly.hv), *Gv = at(a.ly.G), *jm = at(a.ly.jm), *chin = at(a.ly.chin),
         *jb = at(a.ly.jb), *M3 = at(a.ly.M3);
  int* jk = (int*)(lds + a.ly.jk);
  double* Wg = w.W + (long)wk * n * n;
  double* phi = (double*)w.phi + (long)wk * N * Lp;
  const int j = tid & (KP - 1), g = tid / KP;   // column and row group of the n x n and PT passes

  // this thread's basis functions and the two-body parameters
  double4 bf[QL];
  int bk[QL];
#pragma unroll
  for (int q = 0; q < QL; ++q) {
    const int mu = tid + kChainT * q;
    bf[q] = s.bfn[mu < L ? mu : 0];
    bk[q] = s.kind[mu < L ? mu : 0];
  }
  double* j2p = red + 8;
  if (tid < 8) j2p[tid] = s.j2d[tid];
  // state to LDS
  int spin = (a.e0 % N) < n ? 0 : 1;
  for (int q = tid; q < n * n; q += kChainT) {
    const int i = q / n, k = q - i * n;
    B[spin == 0 ? i * ld + k : k * ld + i] = a.Ainv[(long)wk * n * n + q];
  }
  for (int q = tid; q < 3 * N; q += kChainT) r[q] = w.r[(long)wk * 3 * N + q];
  for (int q = tid; q < nn; q += kChainT) {
    nuc[5 * q] = s.R[3 * q]; nuc[5 * q + 1] = s.R[3 * q + 1]; nuc[5 * q + 2] = s.R[3 * q + 2];
    nuc[5 * q + 3] = s.Z[q];
    nuc[5 * q + 4] = s.j1_b[q];
  }
  for (int q = tid; q < N * LJ; q += kChainT) {
    chi[q] = w.chi[(long)wk * N * LJ + q];
    hv[q] = w.hv[(long)wk * N * LJ + q];
  }
  for (int q = tid; q < 2 * LJ; q += kChainT) {
    Gv[q] = w.G3[(long)wk * 2 * LJ + q];
    jm[q] = s.jm[q];
  }
  for (int q = tid; q < LJ; q += kChainT) {
    const double4 f = s.jbfn[q];
    jb[4 * q] = f.x; jb[4 * q + 1] = f.y; jb[4 * q + 2] = f.z; jb[4 * q + 3] = f.w;
    jk[q] = s.jkind[q];
  }
  for (int q = tid; q < 4 * LJ * LJ; q += kChainT) M3[q / (2 * LJ) * (2 * LJ + 1) + q % (2 * LJ)] = s.M3[q];
  double la = w.logabs[wk], sg = w.sign[wk], Jt = w.J[wk];   // kept by thread 0
  int acc_n = 0;
  int since = a.since0, buf = a.buf_spin0, valid = a.valid0, half = -1;
  bool due = false;   // the last move filled the buffer: refresh
  // thread ranges of the set-up: basis functions from thread 0, then the new and
  // the old Jastrow sums and the Jastrow basis from the next waves on
  const int nj = nn + N;
  const int off1 = (L + 63) / 64 * 64, off2 = off1 + (nj + 63) / 64 * 64, off3 = off2 + (nj + 63) / 64 * 64;
  const int t1 = (tid - off1) & (kChainT - 1), t2 = (tid - off2) & (kChainT - 1), t3 = (tid - off3) & (kChainT - 1);

  auto refresh = [&](bool tr) {
    __syncthreads();
    for (int q = tid; q < n * n; q += kChainT) {
      const int i = q / n, k = q - i * n;
      B[i * ld + k] = Wg[q];
    }
    __syncthreads();
    double ldet = 0.0, sdet = 0.0;
    const bool sing = chain_invert<KP>(B, n, ld, tr, prow, ldet, sdet);
    if (tid == 0) {
      la = sing ? -__builtin_inf() : ldet + Jt;
      sg = sdet;
      w.logdet[wk] = ldet;
      w.detsign[wk] = sdet;
      w.singular[wk] = sing ? 1 : 0;
    }
  };
  auto jsum = [&](int t, int e, double px, double py, double pz) {
    double v = 0.0;
    for (int i = t; i < nj; i += kChainT) {
      const bool isn = i < nn;
      const int je = i - nn;
      const double* c = isn ? nuc + 5 * i : r + 3 * je;
      const double dx = px - c[0], dy = py - c[1], dz = pz - c[2];
      const double d = sqrt(dx * dx + dy * dy + dz * dz);
      double f, f1, f2;
      if (isn) {
        if (s.j1_form) { j1_radial(s.j1_form, c[3], c[4], d, f, f1, f2); v += f; }
      } else if (s.j2_form && je != e) {
        j2_radial(s.j2_form, j2p, (e < n) == (je < n), d, f, f1, f2);
        v += f;
      }
    }
    return v;
  };

  for (int t = 0;; ++t) {
    const bool last = t == a.steps;   // only a refresh that is due
    const int e = (int)(((long)a.e0 + t) % N);
    const int sp = last ? buf : (e < n ? 0 : 1), ie = sp == 0 ? e : e - n;
    bool fence = false;   // LDS written since the last barrier
    // the per-move path's schedule
    if (due || (since > 0 && sp != buf)) {
      refresh(sp == 1);
      spin = sp;
      since = 0;
      due = false;
    }
    if (last) break;
    if (sp != spin) {   // nothing buffered: turn the inverse over
      __syncthreads();
      double x[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) x[q] = (g + G * q < n && j < n) ? B[(g + G * q) * ld + j] : 0.0;
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (g + G * q < n && j < n) B[j * ld + g + G * q] = x[q];
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
      for (int q = tid; q < n * (Lp / 2); q += kChainT) {
        const int i = q / (Lp / 2), mu = 2 * (q - i * (Lp / 2));
        const double2 v = *reinterpret_cast<const double2*>((i < nrow ? P + (long)i * Lp : s.Uph + (long)(i - nrow) * Lp) + mu);
        area[mu * np + i] = v.x;
        area[(mu + 1) * np + i] = v.y;
      }
      half = hs;
      fence = true;
    }
    if (t % kChainDraws == 0) {
      __syncthreads();
      for (int q = tid; q < 4 * kChainDraws; q += kChainT) {
        const int k = q >> 2, c = q & 3;
        if (t + k < a.steps)
          draw[q] = c < 3 ? a.disp[((long)(t + k) * Wk + wk) * 3 + c] : a.unif[(long)(t + k) * Wk + wk];
      }
      fence = true;
    }
    if (fence) __syncthreads();

    // set-up: psi(r'), the Jastrow change
    const double* dv = draw + 4 * (t % kChainDraws);
    const double ox = r[3 * e], oy = r[3 * e + 1], oz = r[3 * e + 2];
    const double px = ox + dv[0], py = oy + dv[1], pz = oz + dv[2];
    double sv[QL];
#pragma unroll
    for (int q = 0; q < QL; ++q) {
      const int mu = tid + kChainT * q;
      sv[q] = 0.0;
      if (mu < L) {
        sv[q] = basis_value_rec(bf[q], bk[q], px, py, pz);
        psi[mu] = sv[q];
      }
    }
    double dj = jsum(t1, e, px, py, pz) - jsum(t2, e, ox, oy, oz);
    for (int k = t3; k < LJ; k += kChainT) {
      const double4 f = double4{jb[4 * k], jb[4 * k + 1], jb[4 * k + 2], jb[4 * k + 3]};
      const double v = basis_value_rec(f, jk[k], px, py, pz);
      chin[k] = v;
      dj += (v - chi[e * LJ + k]) * (Gv[sp * LJ + k] - hv[e * LJ + k] + jm[sp * LJ + k]);
    }
    dj = wave_sum(dj);
    if (lane == 0) red[4 * (t & 1) + wave] = dj;
    __syncthreads();

    // the new row (column) of W, its product with the inverse's column
    double x = 0.0;
    if (j < n) {
      int mu = g;
      for (; mu + 3 * G < L; mu += 4 * G) {
        const double p0 = area[mu * np + j], p1 = area[(mu + G) * np + j], p2 = area[(mu + 2 * G) * np + j],
                     p3 = area[(mu + 3 * G) * np + j];
        x += p0 * psi[mu];
        x += p1 * psi[mu + G];
        x += p2 * psi[mu + 2 * G];
        x += p3 * psi[mu + 3 * G];
      }
      for (; mu < L; mu += G) x += area[mu * np + j] * psi[mu];
    }
#pragma unroll
    for (int o = KP; o < 64; o <<= 1) x += __shfl_xor(x, o, 64);
    if (lane < KP) part[wave * 64 + lane] = x;
    __syncthreads();
    double wj = 0.0, cj = 0.0;
    if (lane < n) {
      wj = ((part[lane] + part[64 + lane]) + part[128 + lane]) + part[192 + lane];
      cj = B[lane * ld + ie];
    }
    const double R = wave_sum(wj * cj);
    const double* rd = red + 4 * (t & 1);
    const double dJ = ((rd[0] + rd[1]) + rd[2]) + rd[3];
    const double ratio = R * exp(dJ);
    const bool acc = dv[3] < ratio * ratio;   // uniform
    if (acc) {
      double u = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int i = g + G * q;
        const double wi = __shfl(wj, i & 63, 64);
        if (i < n && j < n) u += wi * B[i * ld + j];
      }
#pragma unroll
      for (int o = KP; o < 64; o <<= 1) u += __shfl_xor(u, o, 64);
      if (lane < KP) pu[wave * 64 + lane] = u;
      if (wave == 0 && lane < n) Wg[sp == 0 ? (long)ie * n + lane : (long)lane * n + ie] = wj;
#pragma unroll
      for (int q = 0; q < QL; ++q) {
        const int mu = tid + kChainT * q;
        if (mu < L) phi[(long)e * Lp + mu] = sv[q];
      }
      for (int o = tid; o < 3 * LJ; o += kChainT) {
        const bool first = o < 2 * LJ;
        const double* row = M3 + (first ? o : sp * LJ + o - 2 * LJ) * (2 * LJ + 1) + sp * LJ;
        double v = 0.0;
        if (first) {
          for (int k = 0; k < LJ; ++k) v += row[k] * (chin[k] - chi[e * LJ + k]);
          Gv[o] += v;
        } else {
          for (int k = 0; k < LJ; ++k) v += row[k] * chin[k];
          hv[e * LJ + o - 2 * LJ] = v;
        }
      }
      __syncthreads();
      if (j < n) {
        u = ((pu[j] + pu[64 + j]) + pu[128 + j]) + pu[192 + j];
        if (j == ie) u -= 1.0;
        u *= 1.0 / R;
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int i = g + G * q;
        const double ci = __shfl(cj, i & 63, 64);
        if (i < n && j < n) B[i * ld + j] = fma(-ci, u, B[i * ld + j]);
      }
      for (int k = tid; k < LJ; k += kChainT) chi[e * LJ + k] = chin[k];
      if (tid == 0) {
        r[3 * e] = px; r[3 * e + 1] = py; r[3 * e + 2] = pz;
        la += log(fabs(R)) + dJ;
        if (R < 0.0) sg = -sg;
        Jt += dJ;
        acc_n += 1;
      }
      __syncthreads();
    }
    valid &= ~(1 << sp);
    since += 1;
    due = since >= a.cap;
  }

  // the walker's state back
  __syncthreads();
  for (int q = tid; q < n * n; q += kChainT) {
    const int i = q / n, k = q - i * n;
    w.A[(long)wk * n * n + q] = B[spin == 0 ? i * ld + k : k * ld + i];
  }
  for (int q = tid; q < 3 * N; q += kChainT) w.r[(long)wk * 3 * N + q] = r[q];
  for (int q = tid; q < N * LJ; q += kChainT) {
    w.chi[(long)wk * N * LJ + q] = chi[q];
    w.hv[(long)wk * N * LJ + q] = hv[q];
  }
  for (int q = tid; q < 2 * LJ; q += kChainT) w.G3[(long)wk * 2 * LJ + q] = Gv[q];
  if (tid == 0) {
    w.logabs[wk] = la;
    w.sign[wk] = sg;
    w.J[wk] = Jt;
    w.wm[wk] = 0;
    if (w.nkeep) w.nkeep[wk] = L;   // the functions a proposal read
    if (a.cnt) a.cnt[wk] += acc_n;
  }
}

// Systems the resident chain takes: FP64 rows, basis functions as orbitals, W
// of at most 64 rows, and a walker's state within 80 KiB of LDS (two
// workgroups per compute unit).
bool chain_ok(const SysDev& s, const WalkDev& w) {
  if (!s.screened() || s.Lq > 0 || s.nu > kChainMaxN || s.L > 2 * kChainT || !w.rpos_P || s.Lp % 32) return false;
  if ((long)s.LJ * s.LJ > 4096 || s.N > 4096 || s.n_nuc > 1024) return false;
  int area;
  return chain_layout(s, area).total <= kChainMaxLds;
}

hipError_t launch_chain(const SysDev& s, const WalkDev& w, int e0, int steps, const double* disp, const double* unif,
                        int32_t* accept_count, int since0, int buf_spin0, int valid0, bool all_rows, const double* Ainv,
                        hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (!chain_ok(s, w) || steps < 1) return hipErrorInvalidValue;
  ChainArgs a{};
  a.e0 = e0; a.steps = steps; a.cap = wb_cap(s); a.since0 = since0; a.buf_spin0 = buf_spin0; a.valid0 = valid0;
  a.all_rows = all_rows ? 1 : 0; a.Ainv = Ainv; a.disp = disp; a.unif = unif; a.cnt = accept_count;
  a.ly = chain_layout(s, a.area_bytes);
  const dim3 grid(w.Wk), blk(kChainT);
#define QMC_CHAIN(K, Q) QMC_LAUNCH_EV((chain_kernel<K, Q>), grid, blk, a.ly.total, st, ev_start, ev_stop, s, w, a)
#define QMC_CHAIN_Q(K) if (s.L <= kChainT) { QMC_CHAIN(K, 1); } else { QMC_CHAIN(K, 2); }
  if (s.nu <= 8) { QMC_CHAIN_Q(8) }
  else if (s.nu <= 16) { QMC_CHAIN_Q(16) }
  else if (s.nu <= 32) { QMC_CHAIN_Q(32) }
  else { QMC_CHAIN_Q(64) }
#undef QMC_CHAIN_Q
#undef QMC_CHAIN
  return hipGetLastError();
}

}  // namespace qmc
