// Basis construction of the prefill stage (Section 3.1.2, Eq. svd): the
// hybrid token sample, token-wise L2 normalisation of the sampled rows (each
// basis group's slice on its own), optional mean-centring, and the top-rank
// right singular vectors of the sampled matrix X [n_s, Dg] per (sequence,
// key/value, basis group).
//
// The right singular vectors of X are the eigenvectors of its Gram matrix
// M = X^T X (centred: X^T X - n_s mu mu^T).  M is formed here in fp64 from the
// stored bf16 rows (64 x 64 output tiles per workgroup, upper triangle only,
// written to both halves).  Of its eigenvectors only those of the `rank`
// largest eigenvalues are wanted, largest first, so the symmetric eigenproblem
// is solved here in fp64 by the textbook route for a few eigenvectors
// (Golub and Van Loan, Matrix Computations, 8.3 and 8.4), for all matrices of
// the call at once:
//   k_tridiag_step  Householder tridiagonalisation M = Q T Q^T, one launch per
//                   column;
//   k_tri_values    the wanted eigenvalues of T by multisection on the Sturm
//                   count, one wave each;
//   k_tri_vectors   their eigenvectors by inverse iteration (LU of T - shift
//                   with partial pivoting), one lane each;
//   k_z_gram, k_z_chol, k_z_solve   their orthonormalisation by a Cholesky
//                   factor of Z^T Z (inverse iteration leaves vectors of close
//                   eigenvalues oblique), repeated where the first pass finds
//                   them far from orthogonal;
//   k_tri_back      Q applied to them.
// The chain of columns bounds it: Dg dependent steps, each a launch, a read of
// what the step before wrote and two block-wide sums (about 5 us).  One 32k
// prompt at Dg = 1024, rank 160 (two matrices): 7.1 ms against 23.5 ms in
// a library solver that computes all eigenvectors by divide and conquer in
// some 4500 launches.
#include <algorithm>
#include <cmath>

#include "s4r_device.h"
#include "s4r_internal.h"

namespace s4r {

constexpr int kGramTile = 64;     // output tile of the Gram kernel
constexpr int kGramChunk = 32;    // samples staged per LDS round
constexpr int kMeanChunks = 32;   // partial column sums (fixed-order merge)

// ---- sampling -------------------------------------------------------------------------
// uniformly spaced early positions (numpy linspace over [0, E - 1], num
// points, rounded half to even), then the recent block [E, T)
__global__ void k_sample_hybrid(int32_t* __restrict__ idx, int64_t T, int n_uniform, int n_recent) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t E = T - n_recent;
  if (i < n_uniform) {
    int64_t v = 0;
    if (n_uniform > 1) {
      if (i == n_uniform - 1) {
        v = E - 1;
      } else {
        const double step = (double)(E - 1) / (double)(n_uniform - 1);
        v = (int64_t)rint((double)i * step);
      }
    }
    idx[i] = (int32_t)v;
  } else if (i < (int64_t)n_uniform + n_recent) {
    idx[i] = (int32_t)(E + (i - n_uniform));
  }
}

// ---- normalisation ----------------------------------------------------------------------
// inv[mat][s] = 1 / ||row slice|| (1 for an all-zero slice); mat = (b * nb + g) * 2 + side.
// One wave per sampled row: grid (ceil(n_s / 4), 2 nb, B), 256 threads.
__global__ __launch_bounds__(256) void k_row_norms(const uint16_t* __restrict__ s_k, const uint16_t* __restrict__ s_v,
                                                   const int32_t* __restrict__ idx, double* __restrict__ inv,
                                                   int64_t n_rows, int n_s, int Dp, int nb) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s = blockIdx.x * 4 + wave;
  const int side = blockIdx.y & 1, g = blockIdx.y >> 1, b = blockIdx.z;
  if (s >= n_s) return;
  const int Dg = Dp / nb;
  const uint16_t* row = (side ? s_v : s_k) + ((int64_t)b * n_rows + idx[s]) * Dp + (int64_t)g * Dg;
  double acc = 0.0;
  for (int d = lane; d < Dg; d += 64) {
    const double x = (double)bf16_bits_to_f32(row[d]);
    acc = fma(x, x, acc);
  }
  for (int o = 32; o > 0; o >>= 1) acc += shfl_xor_d(acc, o);
  if (lane == 0) {
    const int mat = (b * nb + g) * 2 + side;
    inv[(int64_t)mat * n_s + s] = acc > 0.0 ? 1.0 / sqrt(acc) : 1.0;
  }
}

// partial column sums of the normalised samples: part[mat][chunk][d], chunk c
// covering samples c, c + kMeanChunks, ...; grid (Dg / 256, 2 nb * kMeanChunks, B)
__global__ __launch_bounds__(256) void k_col_partial(const uint16_t* __restrict__ s_k, const uint16_t* __restrict__ s_v,
                                                     const int32_t* __restrict__ idx, const double* __restrict__ inv,
                                                     double* __restrict__ part, int64_t n_rows, int n_s, int Dp,
                                                     int nb) {
  const int d = blockIdx.x * 256 + threadIdx.x;
  const int sg = blockIdx.y / kMeanChunks, c = blockIdx.y % kMeanChunks;
  const int side = sg & 1, g = sg >> 1, b = blockIdx.z;
  const int Dg = Dp / nb;
  const int mat = (b * nb + g) * 2 + side;
  const uint16_t* base = (side ? s_v : s_k) + (int64_t)b * n_rows * Dp + (int64_t)g * Dg + d;
  double acc = 0.0;
  for (int s = c; s < n_s; s += kMeanChunks)
    acc = fma((double)bf16_bits_to_f32(base[(int64_t)idx[s] * Dp]), inv[(int64_t)mat * n_s + s], acc);
  part[((int64_t)mat * kMeanChunks + c) * Dg + d] = acc;
}

// ---- Gram matrix --------------------------------------------------------------------------
// M[mat] (column-major Dg x Dg) = sum_s xh_s xh_s^T (- n_s mu mu^T when centred).
// Grid (T (T + 1) / 2 upper tiles, 2 nb, B) with T = Dg / 64; 256 threads.
// The samples of a round (32 of them, both 64-column ranges, weighted by the
// row norms' inverses) are staged in LDS as fp64, the next round's requested
// while the current one is multiplied; wave w accumulates the
// 32 x 32 quadrant (w / 2, w % 2) of the tile on the fp64 matrix cores
// (16x16x4: lane l holds A[row l % 16][sample l / 16] and B[sample l / 16]
// [column l % 16], and receives D rows l / 16 + 4 i of column l % 16, as
// probed on gfx950), four 16 x 16 blocks per wave, four samples per step.
typedef double double4_t __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_gram(const uint16_t* __restrict__ s_k, const uint16_t* __restrict__ s_v,
                                              const int32_t* __restrict__ idx, const double* __restrict__ inv,
                                              const double* __restrict__ part, double* __restrict__ M,
                                              int64_t n_rows, int n_s, int Dp, int nb, int center) {
  const int Dg = Dp / nb;
  const int nt = Dg / kGramTile;
  // upper-triangle tile (ti <= tj) of linear index blockIdx.x
  int ti = 0, rem = blockIdx.x;
  while (rem >= nt - ti) {
    rem -= nt - ti;
    ++ti;
  }
  const int tj = ti + rem;
  const int side = blockIdx.y & 1, g = blockIdx.y >> 1, b = blockIdx.z;
  const int mat = (b * nb + g) * 2 + side;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int lr = lane & 15, lk = lane >> 4;       // MFMA operand row / column, sample within the step
  const int qr = (wave >> 1) * 32, qc = (wave & 1) * 32;   // the wave's quadrant
  const uint16_t* base = (side ? s_v : s_k) + (int64_t)b * n_rows * Dp + (int64_t)g * Dg;
  const double* inv_m = inv + (int64_t)mat * n_s;
  __shared__ double xa[kGramChunk][kGramTile + 1], xb[kGramChunk][kGramTile + 1];
  double4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int i0 = ti * kGramTile, j0 = tj * kGramTile;
  // the next round's sample values are requested before this round's MFMAs
  // run and written to LDS after them (8 per thread and column range: sample
  // wave + 4 k, column lane); the round after's positions are read with them,
  // so a round waits for one memory latency and not for two in a row (955 ->
  // 618 us for two matrices of 6553 samples at Dg = 1024)
  constexpr int kPer = kGramChunk * kGramTile / 256;
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  uint16_t ra[kPer], rb[kPer];
  double rw[kPer], nw[kPer];
  int32_t nid[kPer];
  auto positions = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int s = min(s0 + wv + 4 * k, n_s - 1);
      nid[k] = idx[s];
      nw[k] = inv_m[s];
    }
  };
  auto fetch = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint16_t* row = base + (int64_t)nid[k] * Dp + lane;
      ra[k] = row[i0];
      rb[k] = row[j0];
      rw[k] = s0 + wv + 4 * k < n_s ? nw[k] : 0.0;
    }
    positions(s0 + kGramChunk);
  };
  auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int r = wv + 4 * k, col = lane;
      xa[r][col] = (double)bf16_bits_to_f32(ra[k]) * rw[k];
      xb[r][col] = (double)bf16_bits_to_f32(rb[k]) * rw[k];
    }
  };
  positions(0);
  fetch(0);
  stage();
  __syncthreads();
  for (int s0 = 0; s0 < n_s; s0 += kGramChunk) {
    if (s0 + kGramChunk < n_s) fetch(s0 + kGramChunk);
#pragma unroll
    for (int k4 = 0; k4 < kGramChunk; k4 += 4) {
      double a[2], bb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = xa[k4 + lk][qr + 16 * i + lr];
#pragma unroll
      for (int j = 0; j < 2; ++j) bb[j] = xb[k4 + lk][qc + 16 * j + lr];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], bb[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
    if (s0 + kGramChunk < n_s) {
      stage();
      __syncthreads();
    }
  }
  double* Mm = M + (int64_t)mat * Dg * Dg;
  const double* pm = part + (int64_t)mat * kMeanChunks * Dg;
  const double inv_n = 1.0 / (double)n_s;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int gj = j0 + qc + 16 * j + lr;
    double mj = 0.0;
    if (center)
      for (int c = 0; c < kMeanChunks; ++c) mj += pm[(int64_t)c * Dg + gj];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int gi = i0 + qr + 16 * i + lk + 4 * e;
        double v = acc[i][j][e];
        if (center) {
          double mi = 0.0;
          for (int c = 0; c < kMeanChunks; ++c) mi += pm[(int64_t)c * Dg + gi];
          v -= (mi * inv_n) * (mj * inv_n) * (double)n_s;
        }
        Mm[gi + (int64_t)gj * Dg] = v;
        Mm[gj + (int64_t)gi * Dg] = v;
      }
  }
}

// ---- tridiagonalisation ---------------------------------------------------------------------
// Step j of M = Q T Q^T, Q = H_0 H_1 .., H_j = I - tau_j v_j v_j^T with v_j[c] =
// 0 for c <= j and v_j[j + 1] = 1.  Grid (n / 8, matrices), 256 threads, NC =
// n / 256: workgroup x owns rows 8 x .. 8 x + 7, thread t columns t + 256 i.
// Every workgroup forms for itself, from the previous step's v and y = A v
// (buffers of the step's parity), the rank-2 update's w = tau y - kappa v, the
// updated column j and from it this step's reflector; then it updates its own
// rows, A -= v w^T + w v^T, and multiplies them with the new v while they are
// in registers.  So a column costs one launch, nothing is exchanged within it,
// and a workgroup's rows are requested before the chain of sums begins.  The
// last workgroup records d, e, tau and v, and puts the previous v into row
// j - 1 of A, which no step reads any more.
constexpr int kTriRows = 8;

struct TriState {
  double* A;      // [matrices][n][n]
  double* v;      // [matrices][2][n]
  double* y;      // [matrices][2][n]
  double* d;      // [matrices][n]
  double* e;      // [matrices][n]
  double* tau;    // [matrices][n]
};

__device__ __forceinline__ double block_sum4(double x, double* s) {
  x = wave_sum(x);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = x;
  lds_barrier();
  return (s[0] + s[1]) + (s[2] + s[3]);
}

template <int NC>
__global__ __launch_bounds__(256) void k_tridiag_step(TriState S, int j) {
  constexpr int n = NC * 256;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int row0 = blockIdx.x * kTriRows;
  const bool record = blockIdx.x == gridDim.x - 1;
  if (row0 + kTriRows <= j + 1 && !record) return;
  const int64_t mat = blockIdx.y;
  double* A = S.A + mat * n * n;
  const double* vp_ = S.v + (mat * 2 + ((j + 1) & 1)) * n;   // the previous step's
  const double* yp_ = S.y + (mat * 2 + ((j + 1) & 1)) * n;
  double* vn_ = S.v + (mat * 2 + (j & 1)) * n;
  double* yn_ = S.y + (mat * 2 + (j & 1)) * n;
  __shared__ double s1[4], s2[4], red[4][kTriRows];

  double vp[NC], yp[NC], col[NC], a[kTriRows][NC];
  const bool first = j == 0;                       // no previous reflector (uniform)
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = t + 256 * i;
    col[i] = A[(int64_t)j * n + c];
    vp[i] = first ? 0.0 : vp_[c];
    yp[i] = (first || c < j) ? 0.0 : yp_[c];       // (y is set from the previous step's column on)
  }
  const int j1 = min(j + 1, n - 1);
  double vr[kTriRows], yr[kTriRows];
#pragma unroll
  for (int r = 0; r < kTriRows; ++r) {
    const int row = max(row0 + r, j1);             // finished rows repeat row j + 1 and are not stored
#pragma unroll
    for (int i = 0; i < NC; ++i) a[r][i] = A[(int64_t)row * n + t + 256 * i];
    vr[r] = first ? 0.0 : vp_[row];
    yr[r] = first ? 0.0 : yp_[row];
  }
  const double tau = first ? 0.0 : S.tau[mat * n + j - 1];
  const double vj = first ? 0.0 : 1.0, yj = first ? 0.0 : yp_[j];
  const double vj1 = first ? 0.0 : vp_[j1], yj1 = first ? 0.0 : yp_[j1];
  const double ajj = A[(int64_t)j * n + j], ajj1 = A[(int64_t)j * n + j1];

  // w = tau y - kappa v with kappa = tau^2 (v . y) / 2, then column j as updated
  double dot = 0.0;
#pragma unroll
  for (int i = 0; i < NC; ++i) dot = fma(vp[i], yp[i], dot);
  dot = block_sum4(dot, s1);
  const double kap = 0.5 * tau * tau * dot;
  const double wj = fma(tau, yj, -kap * vj), wj1 = fma(tau, yj1, -kap * vj1);
  double w[NC], xn = 0.0;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    w[i] = fma(tau, yp[i], -kap * vp[i]);
    col[i] = fma(-wj, vp[i], fma(-vj, w[i], col[i]));
    const double x = t + 256 * i > j + 1 ? col[i] : 0.0;
    xn = fma(x, x, xn);
  }
  xn = block_sum4(xn, s2);
  const double dj = ajj - 2.0 * vj * wj;
  const double al = fma(-wj, vj1, fma(-vj, wj1, ajj1));
  double beta = al, tn = 0.0, scale = 0.0;
  if (xn != 0.0) {                                 // (also a NaN: it goes on into every result)
    beta = -copysign(sqrt(fma(al, al, xn)), al);
    tn = (beta - al) / beta;
    scale = 1.0 / (al - beta);
  }
  double vn[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = t + 256 * i;
    vn[i] = c > j + 1 ? col[i] * scale : (c == j + 1 ? 1.0 : 0.0);
  }
  if (record) {
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      vn_[t + 256 * i] = vn[i];
      if (!first) A[(int64_t)(j - 1) * n + t + 256 * i] = vp[i];
    }
    if (t == 0) {
      S.d[mat * n + j] = dj;
      S.e[mat * n + j] = j < n - 1 ? beta : 0.0;
      S.tau[mat * n + j] = tn;
    }
  }
  // this workgroup's rows: update, and their products with the new v
  double p[kTriRows];
#pragma unroll
  for (int r = 0; r < kTriRows; ++r) {
    const double wr = fma(tau, yr[r], -kap * vr[r]);
    p[r] = 0.0;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const double x = fma(-wr, vp[i], fma(-vr[r], w[i], a[r][i]));
      if (row0 + r > j && t + 256 * i > j) A[(int64_t)(row0 + r) * n + t + 256 * i] = x;
      p[r] = fma(x, vn[i], p[r]);
    }
  }
  // eight sums over the wave: lane swaps that halve the values a lane holds,
  // then the 16 lanes of a row; rows 0 .. 3 of the wave end with p0 p2 p1 p3
  const double z0 = swap16_add(swap32_add(p[0], p[1]), swap32_add(p[2], p[3]));
  const double z1 = swap16_add(swap32_add(p[4], p[5]), swap32_add(p[6], p[7]));
  auto row_sum = [](double x) {
    x += dpp_d<0xB1>(x);
    x += dpp_d<0x4E>(x);
    x += dpp_d<0x124>(x);
    x += dpp_d<0x128>(x);
    return x;
  };
  const double q0 = row_sum(z0), q1 = row_sum(z1);
  if ((lane & 15) == 0) {
    const int g = lane >> 4, m = (g >> 1) | ((g & 1) << 1);
    red[wave][m] = q0;
    red[wave][4 + m] = q1;
  }
  lds_barrier();
  if (t < kTriRows && row0 + t > j) yn_[row0 + t] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
}

// ---- eigenvalues of T -------------------------------------------------------------------------
// The q-th largest eigenvalue of T, q < r: one wave each, grid (ceil(r / 4),
// matrices).  Every sweep evaluates the Sturm count (eigenvalues below x: sign
// changes of the leading minors' recurrence p_{i+1} = (d_i - x) p_i - e_i^2
// p_{i-1}, rescaled every four terms) at 64 points of the interval, so ten
// sweeps narrow Gershgorin's interval by 65^10 = 2^60.  T is scaled to norm 1;
// e^2 is kept above 1e-40 so a split of T (e = 0) needs no special case.
// info[mat] = 1 where T is not finite.
__global__ __launch_bounds__(256) void k_tri_values(const double* __restrict__ d_all, const double* __restrict__ e_all,
                                                    double* __restrict__ lam, double* __restrict__ norm,
                                                    int32_t* __restrict__ info, int n, int rk, int rv, int rmax) {
  const int64_t mat = blockIdx.y;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int r = (mat & 1) == 0 ? rk : rv;          // keys, values
  __shared__ double ds[2048 + 16], es[2048 + 16], sn[4];
  const double* d = d_all + mat * n;
  const double* e = e_all + mat * n;
  double bound = 0.0;
  bool finite = true;
  for (int i = t; i < n; i += 256) {
    const double di = d[i], ei = e[i], em = i > 0 ? e[i - 1] : 0.0;
    ds[i] = di;
    es[i] = ei;
    const double g = fabs(di) + fabs(ei) + fabs(em);
    finite = finite && g < INFINITY;               // false for a NaN too
    bound = fmax(bound, g);
  }
  for (int o = 32; o > 0; o >>= 1) bound = fmax(bound, shfl_xor_d(bound, o));
  if (lane == 0) sn[wave] = bound;
  const int bad = __syncthreads_or(!finite);
  bound = fmax(fmax(sn[0], sn[1]), fmax(sn[2], sn[3]));
  const double nrm = bound > 0.0 ? bound : 1.0, inv = 1.0 / nrm;
  if (blockIdx.x == 0 && t == 0) {
    norm[mat] = nrm;
    info[mat] = bad ? 1 : 0;
  }
  __syncthreads();
  for (int i = t; i < n; i += 256) {
    const double x = es[i] * inv;
    ds[i] *= inv;
    es[i] = fmax(x * x, 1e-40);
  }
  if (t < 16) ds[n + t] = es[n + t] = 0.0;
  __syncthreads();
  const int q = blockIdx.x * 4 + wave;
  if (q >= r || bad) return;
  const int m = n - 1 - q;                         // its index from the smallest
  double lo = -1.0 - 1e-15, hi = 1.0 + 1e-15;
  for (int it = 0; it < 10; ++it) {
    const double x = lo + (hi - lo) * ((double)(lane + 1) * (1.0 / 65.0));
    double pa = 1.0, pb = ds[0] - x;
    int below = (int)((uint32_t)__double2hiint(pb) >> 31);
    // terms 1 .. n - 1 in blocks of eight, the next block's read ahead (past
    // the end: zeros, whose terms are not counted)
    double dn[8], en[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      dn[u] = ds[1 + u];
      en[u] = es[u];
    }
    for (int i = 1; i < n; i += 8) {
      double dc[8], ec[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        dc[u] = dn[u];
        ec[u] = en[u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        dn[u] = ds[i + 8 + u];
        en[u] = es[i + 7 + u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double pc = fma(dc[u] - x, pb, -ec[u] * pa);
        const int change = (int)((uint32_t)(__double2hiint(pc) ^ __double2hiint(pb)) >> 31);
        below += i + u < n ? change : 0;
        pa = pb;
        pb = pc;
        if (u % 4 == 3) {
          // both scaled by the power of two that brings the larger near 1
          const uint32_t ea = (uint32_t)__double2hiint(pa) & 0x7FF00000u, eb = (uint32_t)__double2hiint(pb) & 0x7FF00000u;
          const double sc = __hiloint2double((int)(0x7FE00000u - min(max(max(ea, eb), 0x00100000u), 0x7FD00000u)), 0);
          pa *= sc;
          pb *= sc;
        }
      }
    }
    const uint64_t over = __ballot(below > m);     // points above the eigenvalue
    const int f = over ? __ffsll((unsigned long long)over) - 1 : 64;
    const double step = (hi - lo) * (1.0 / 65.0), base = lo;
    if (f < 64) hi = base + step * (double)(f + 1);
    if (f > 0) lo = base + step * (double)f;
  }
  if (lane == 0) lam[mat * rmax + q] = 0.5 * (lo + hi);   // of T / norm
}

// ---- eigenvectors of T ------------------------------------------------------------------------
// Inverse iteration, one lane per eigenvalue: EV = 2048 / n of them per
// workgroup (one wave; T and the factors of its lanes in LDS, so the serial
// sweeps over n run at LDS latency).  LU of T / norm - (lambda + kShift) with
// partial pivoting, a start vector of its own, two solves (the first by U alone).
//
// Eigenvalues may coincide to rounding: repeated or orthogonal rows, equal
// blocks, the zeros of a prompt with few distinct rows.  At the eigenvalue
// itself a solve would magnify most whichever member of the cluster rounding
// puts nearest, the same one in every lane.  kShift keeps all of them at about
// the same distance, some 500 times the rounding of T's norm, so a cluster's
// vectors are its starts projected on its space and stay independent; two
// solves leave a neighbour at a gap g (1 = the norm) with (kShift / g)^2 of
// its start: 1e-14 at 1e-6, and a mixture below 1e-12 costs no more energy
// than the gap.  In clusters, block and projection matrices and graded spectra
// of 256 to 1024 columns the smallest pivot of the Cholesky factor is 1e-4 at
// the median and 1e-12 at worst with two solves, lost altogether in one
// of a hundred with three (and at the eigenvalue itself in most).
constexpr double kShift = 1.1368683772161603e-13;   // 2^-43

// orthonormalisation rounds per matrix, what each leaves in
// state[mat] = 4 round + code, and the pivots that decide: 1 is a unit vector
// orthogonal to those before it, and the factor's error grows with its inverse
constexpr int kOrthoRounds = 3;
enum OrthoCode { kOrthoDone = 0, kOrthoAgain = 1, kOrthoLost = 2 };   // Lost: other start vectors
constexpr double kPivAgain = 1e-3, kPivLost = 1e-12;
// whether matrix mat takes part in a round, given the code the round before left
__device__ __forceinline__ bool ortho_active(const int32_t* info, const int32_t* state, int64_t mat, int round,
                                             int code) {
  return info[mat] == 0 && (round == 0 || (state[mat] & 3) >= code);
}

// component i of start vector q of a round, in [-1, 1): the index times the
// bits of the golden ratio plus the vector's times those of sqrt(2), folded
// and multiplied again so that different q share no pattern
__device__ __forceinline__ double start_component(int i, int q, int round) {
  constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull, kRoot2 = 0x6A09E667F3BCC909ull;
  uint64_t h = (uint64_t)(i + 1) * kGolden + (uint64_t)(q + 1 + 4096 * round) * kRoot2;
  h = (h ^ (h >> 32)) * kGolden;
  h = (h ^ (h >> 29)) * kRoot2;
  return (double)(int64_t)h * (1.0 / 9223372036854775808.0);
}

__global__ __launch_bounds__(64) void k_tri_vectors(const double* __restrict__ d_all, const double* __restrict__ e_all,
                                                    const double* __restrict__ lam, const double* __restrict__ norm,
                                                    const int32_t* __restrict__ info,
                                                    const int32_t* __restrict__ state, double* __restrict__ Z, int n,
                                                    int rk, int rv, int rmax, int ev, int round) {
  const int64_t mat = blockIdx.y;
  const int lane = threadIdx.x;
  const int r = (mat & 1) == 0 ? rk : rv;
  if (!ortho_active(info, state, mat, round, kOrthoLost)) return;
  __shared__ double ds[2048 + 16], es[2048 + 16];
  __shared__ double li[2048], pi[2048], u1[2048], u2[2048], xs[2048];   // [k][ev]
  __shared__ uint8_t sw[2048];
  const int q0 = blockIdx.x * ev;
  if (q0 >= r) return;
  const double inv = 1.0 / norm[mat];
  for (int i = lane; i < n; i += 64) {
    ds[i] = d_all[mat * n + i] * inv;
    es[i] = e_all[mat * n + i] * inv;
  }
  if (lane < 16) ds[n + lane] = es[n + lane] = 0.0;
  for (int i = lane; i < n * ev; i += 64) xs[i] = start_component(i / ev, q0 + i % ev, round);
  lds_barrier();
  const int q = min(q0 + lane, r - 1);
  if (lane < ev) {
    constexpr double kTiny = 2.2e-16;              // smallest pivot, for a norm of 1
    const double x = lam[mat * rmax + q] + kShift;
    auto at = [&](int k) { return k * ev + lane; };
    double b = ds[0] - x, c = es[0];
    for (int k0 = 0; k0 < n; k0 += 8) {             // (n is a multiple of 256; T has zeros after its end)
      double sb[9], dg[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        sb[u] = es[k0 + u];
        dg[u] = ds[k0 + u + 1];
      }
      sb[8] = es[k0 + 8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = k0 + u;
        // row k + 1: (sub, dn, en); none after the last row
        const bool more = k + 1 < n;
        const double sub = sb[u], dn = dg[u] - x, en = sb[u + 1];
        const bool swap = more && fabs(b) < fabs(sub);
        double piv = swap ? sub : b;
        if (fabs(piv) < kTiny) piv = copysign(kTiny, piv);
        const double rp = 1.0 / piv;
        const double l = more ? (swap ? b : sub) * rp : 0.0;
        li[at(k)] = l;
        pi[at(k)] = rp;
        u1[at(k)] = more ? (swap ? dn : c) : 0.0;
        u2[at(k)] = swap ? en : 0.0;
        sw[at(k)] = swap ? 1 : 0;
        b = swap ? fma(-l, dn, c) : fma(-l, c, dn);
        c = swap ? -l * en : en;
      }
    }
    double sc = 1.0;                               // applied when a sweep reads x
    for (int it = 0; it < 2; ++it) {
      if (it > 0) {                                // x = L^-1 P x
        double cur = xs[at(0)] * sc;
        for (int k0 = 0; k0 + 1 < n; k0 += 8) {
          double nx[8], l[8];
          int s[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int k = min(k0 + u, n - 2);
            nx[u] = xs[at(k + 1)];
            l[u] = li[at(k)];
            s[u] = sw[at(k)];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if (k0 + u + 1 < n) {
              const double y = nx[u] * sc;
              const double top = s[u] ? y : cur, bot = s[u] ? cur : y;
              xs[at(k0 + u)] = top;
              cur = fma(-l[u], top, bot);
            }
          }
        }
        xs[at(n - 1)] = cur;
      }
      double x1 = 0.0, x2 = 0.0, mx = 0.0;          // x = U^-1 x
      for (int k0 = n - 1; k0 >= 0; k0 -= 8) {
        double y[8], p[8], a1[8], a2[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int k = max(k0 - u, 0);
          y[u] = xs[at(k)];
          p[u] = pi[at(k)];
          a1[u] = u1[at(k)];
          a2[u] = u2[at(k)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const double z = fma(-a1[u], x1, fma(-a2[u], x2, y[u])) * p[u];
          if (k0 - u >= 0) {
            xs[at(k0 - u)] = z;
            x2 = x1;
            x1 = z;
            mx = fmax(mx, fabs(z));
          }
        }
      }
      sc = mx > 0.0 ? 1.0 / mx : 1.0;
    }
    double ss = 0.0;
    for (int k = 0; k < n; ++k) {
      const double y = xs[at(k)] * sc;
      ss = fma(y, y, ss);
    }
    ds[lane] = sc / sqrt(ss);                      // (T is no longer needed)
  }
  lds_barrier();
  for (int i = lane; i < n * ev; i += 64) {
    const int l = i / n, k = i % n;
    if (q0 + l < r) Z[(mat * rmax + q0 + l) * n + k] = xs[k * ev + l] * ds[l];
  }
}

// ---- orthonormalisation -----------------------------------------------------------------------
// G = Z Z^T over the r vectors (rows of Z, length n), lower tiles of 16 x 16:
// grid (tiles, matrices), thread (a, b) one element
__global__ __launch_bounds__(256) void k_z_gram(const double* __restrict__ Z, double* __restrict__ G,
                                                const int32_t* __restrict__ info, const int32_t* __restrict__ state,
                                                int n, int rk, int rv, int rmax, int round) {
  const int64_t mat = blockIdx.y;
  const int r = (mat & 1) == 0 ? rk : rv;
  if (!ortho_active(info, state, mat, round, kOrthoAgain)) return;
  int ta = 0, rem = blockIdx.x;
  while (rem > ta) {
    rem -= ta + 1;
    ++ta;
  }
  const int tb = rem, t = threadIdx.x, a = t >> 4, b = t & 15;
  if (ta * 16 >= r) return;
  __shared__ double za[16][65], zb[16][65];
  const double* Zm = Z + mat * rmax * n;
  double acc = 0.0;
  for (int k0 = 0; k0 < n; k0 += 64) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = t + 256 * u, row = i >> 6, k = i & 63;
      za[row][k] = Zm[(int64_t)min(ta * 16 + row, r - 1) * n + k0 + k];
      zb[row][k] = Zm[(int64_t)min(tb * 16 + row, r - 1) * n + k0 + k];
    }
    __syncthreads();
#pragma unroll 16
    for (int k = 0; k < 64; ++k) acc = fma(za[a][k], zb[b][k], acc);
    __syncthreads();
  }
  if (ta * 16 + a < r && tb * 16 + b < r) G[(mat * rmax + ta * 16 + a) * rmax + tb * 16 + b] = acc;
}

// Cholesky factor of G, one workgroup per matrix (four quarters of the inner
// sum per row): L row-major over G's lower triangle in place, its diagonal as
// the reciprocal; the columns already found are read from LDS (column j from
// its diagonal down) up to kCholLds vectors, else from LT in memory.  Its
// smallest pivot decides whether the matrix needs another round (a NaN among
// the vectors counts as lost)
constexpr int kCholLds = 180;
template <bool LDS>
__global__ __launch_bounds__(1024) void k_z_chol(double* __restrict__ G, double* __restrict__ LT,
                                                 const int32_t* __restrict__ info, int32_t* __restrict__ state, int rk,
                                                 int rv, int rmax, int round) {
  const int64_t mat = blockIdx.x;
  const int r = (mat & 1) == 0 ? rk : rv;
  if (!ortho_active(info, state, mat, round, kOrthoAgain)) return;
  const int i = threadIdx.x & 255, qr = threadIdx.x >> 8;
  double* Gm = G + mat * rmax * rmax;
  double* Lm = LT + mat * rmax * rmax;
  __shared__ double red[4][256], s_piv;
  int code = kOrthoDone;                           // uniform: every thread reads every pivot
  __shared__ double lc[LDS ? kCholLds * (kCholLds + 1) / 2 : 1];
  auto col = [&](int j) { return j * r - j * (j - 1) / 2 - j; };   // L[i][j] at lc[col(j) + i]
  for (int k = 0; k < r; ++k) {
    double acc = 0.0;
    if (i >= k && i < r) {
#pragma unroll 8
      for (int j = qr; j < k; j += 4) {
        if constexpr (LDS)
          acc = fma(lc[col(j) + i], lc[col(j) + k], acc);
        else
          acc = fma(Lm[(int64_t)j * rmax + i], Lm[(int64_t)j * rmax + k], acc);
      }
    }
    red[qr][i] = acc;
    const double gik = qr == 0 && i >= k && i < r ? Gm[(int64_t)i * rmax + k] : 0.0;
    __syncthreads();
    const double s = gik - ((red[0][i] + red[1][i]) + (red[2][i] + red[3][i]));
    if (qr == 0 && i == k) s_piv = s;
    __syncthreads();
    const double piv = s_piv;
    if (!(piv > kPivLost)) {
      code = kOrthoLost;
      break;
    }
    code = piv < kPivAgain ? kOrthoAgain : code;
    if (qr == 0 && i >= k && i < r) {
      const double ip = 1.0 / sqrt(piv), v = s * ip;
      Gm[(int64_t)i * rmax + k] = i == k ? ip : v;
      if constexpr (LDS)
        lc[col(k) + i] = v;
      else
        Lm[(int64_t)k * rmax + i] = v;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) state[mat] = 4 * round + code;
}

// Z <- L^-1 Z where this round found a factor: every component of the vectors
// on its own, grid (n / 64, matrices), lane = component
__global__ __launch_bounds__(64) void k_z_solve(double* __restrict__ Z, const double* __restrict__ G,
                                                const int32_t* __restrict__ info, const int32_t* __restrict__ state,
                                                int n, int rk, int rv, int rmax, int round) {
  const int64_t mat = blockIdx.y;
  const int r = (mat & 1) == 0 ? rk : rv;
  if (info[mat] || (state[mat] >> 2) != round || (state[mat] & 3) == kOrthoLost) return;
  __shared__ double z[256][64];
  const int lane = threadIdx.x;
  double* Zm = Z + mat * rmax * n + blockIdx.x * 64 + lane;
  const double* L = G + mat * rmax * rmax;
  for (int k = 0; k < r; ++k) z[k][lane] = Zm[(int64_t)k * n];
  for (int k = 0; k < r; ++k) {
    double acc0 = z[k][lane], acc1 = 0.0;
    int j = 0;
    for (; j + 8 <= k; j += 8) {
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        acc0 = fma(-L[(int64_t)k * rmax + j + u], z[j + u][lane], acc0);
        acc1 = fma(-L[(int64_t)k * rmax + j + u + 1], z[j + u + 1][lane], acc1);
      }
    }
    for (; j < k; ++j) acc0 = fma(-L[(int64_t)k * rmax + j], z[j][lane], acc0);
    const double x = (acc0 + acc1) * L[(int64_t)k * rmax + k];
    z[k][lane] = x;
    Zm[(int64_t)k * n] = x;
  }
}

// ---- Q applied to the vectors -------------------------------------------------------------------
// x <- H_0 (H_1 (.. x)), one wave per vector with x in registers; v_j is row j
// of A, the next three requested ahead; grid (ceil(r / 4), matrices)
template <int NC>
__global__ __launch_bounds__(256, 1) void k_tri_back(TriState S, double* __restrict__ Z, int rk, int rv, int rmax) {
  constexpr int n = NC * 256, NP = NC * 2;         // pairs of components per lane
  const int64_t mat = blockIdx.y;
  const int r = (mat & 1) == 0 ? rk : rv;
  const int lane = threadIdx.x & 63, q = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= r) return;
  const double2* V = reinterpret_cast<const double2*>(S.A + mat * n * n) + lane;
  const double* tau = S.tau + mat * n;
  double2* zp = reinterpret_cast<double2*>(Z + (mat * rmax + q) * n) + lane;
  double2 x[NP], v0[NP], v1[NP], v2[NP], v3[NP];
  double t0, t1, t2, t3;
  // reflectors past the first read row 0 with tau = 0
  auto load = [&](int j, double2 (&v)[NP], double& t) __attribute__((always_inline)) {
    const int jc = max(j, 0);
#pragma unroll
    for (int i = 0; i < NP; ++i) v[i] = V[(int64_t)jc * (n / 2) + 64 * i];
    t = j >= 0 ? tau[jc] : 0.0;
  };
  auto apply = [&](const double2 (&v)[NP], double t) __attribute__((always_inline)) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      s0 = fma(v[i].x, x[i].x, s0);
      s1 = fma(v[i].y, x[i].y, s1);
    }
    const double f = -t * wave_sum(s0 + s1);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      x[i].x = fma(f, v[i].x, x[i].x);
      x[i].y = fma(f, v[i].y, x[i].y);
    }
  };
#pragma unroll
  for (int i = 0; i < NP; ++i) x[i] = zp[64 * i];
  load(n - 3, v0, t0);
  load(n - 4, v1, t1);
  load(n - 5, v2, t2);
  for (int j = n - 3; j >= 0; j -= 4) {
    load(j - 3, v3, t3);
    apply(v0, t0);
    load(j - 4, v0, t0);
    apply(v1, t1);
    load(j - 5, v1, t1);
    apply(v2, t2);
    load(j - 6, v2, t2);
    apply(v3, t3);
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) zp[64 * i] = x[i];
}

// ---- bases ----------------------------------------------------------------------------------
// bases[b][g][d][c] = component d of vector c (largest eigenvalue first) of
// matrix (b * nb + g) * 2 + side, in the storage format, for the configured
// rank's columns c < rank_*; the padding columns up to the storage width
// (stride_*) are zero.  A matrix that is not finite (info != 0), or whose
// vectors were lost in every round, gets quiet-NaN bases, so the failure
// reaches the caller.
template <typename T>
__global__ __launch_bounds__(256) void k_write_bases(const double* __restrict__ Z, const int32_t* __restrict__ info,
                                                     const int32_t* __restrict__ state, T* __restrict__ bases_k, T* __restrict__ bases_v, int B, int nb,
                                                     int Dg, int stride_k, int stride_v, int rank_k, int rank_v,
                                                     int rmax) {
  const int side = blockIdx.y;
  const int stride = side ? stride_v : stride_k, rank = side ? rank_v : rank_k;
  const int64_t n = (int64_t)B * nb * Dg * stride;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % stride);
    const int d = (int)((e / stride) % Dg);
    const int64_t bg = e / ((int64_t)stride * Dg);
    const int64_t mat = bg * 2 + side;
    const double v = c < rank ? Z[(mat * rmax + c) * Dg + d] : 0.0;
    store_elem(side ? bases_v : bases_k, e, info[mat] == 0 && (state[mat] & 3) != kOrthoLost ? v : __builtin_nan(""));
  }
}

// ---- host side -----------------------------------------------------------------------------

void bases_sample_counts(int64_t T, double eta, int* n_uniform, int* n_recent) {
  const int64_t n = std::max<int64_t>(1, (int64_t)std::floor(eta * (double)T));
  const int64_t nr = std::min<int64_t>(T, (int64_t)std::nearbyint(0.7 * (double)n));
  const int64_t nu = n - nr;
  const int64_t E = T - nr;
  *n_recent = (int)nr;
  *n_uniform = (nu > 0 && E > 0) ? (int)std::min<int64_t>(nu, E) : 0;
}

namespace {
struct BasesLayout {
  size_t m, v, y, d, e, tau, lam, norm, info, state, z, g, lt, inv, part, idx, total;
};
BasesLayout bases_layout(const Problem& P, int n_s) {
  const size_t nmat = (size_t)P.B * 2 * P.nb, Dg = P.Dg, r = std::max(P.rank_cfg, P.rank_v_cfg);
  BasesLayout l;
  size_t o = 0;
  auto put = [&](size_t& at, size_t bytes) {
    at = o;
    o = (o + bytes + 255) & ~(size_t)255;
  };
  put(l.m, nmat * Dg * Dg * 8);
  put(l.v, nmat * 2 * Dg * 8);
  put(l.y, nmat * 2 * Dg * 8);
  put(l.d, nmat * Dg * 8);
  put(l.e, nmat * Dg * 8);
  put(l.tau, nmat * Dg * 8);
  put(l.lam, nmat * r * 8);
  put(l.norm, nmat * 8);
  put(l.info, nmat * 4);
  put(l.state, nmat * 4);
  put(l.z, nmat * r * Dg * 8);
  put(l.g, nmat * r * r * 8);
  put(l.lt, nmat * r * r * 8);
  put(l.inv, nmat * (size_t)n_s * 8);
  put(l.part, nmat * kMeanChunks * Dg * 8);
  put(l.idx, (size_t)n_s * 4);
  l.total = o;
  return l;
}

template <int NC>
void launch_eigen(const TriState& S, double* lam, double* norm, int32_t* info, int32_t* state, double* Z, double* G,
                  double* LT, int nmat, int rk, int rv, hipStream_t st) {
  constexpr int n = NC * 256;
  const int rmax = std::max(rk, rv), ev = 2048 / n;
  for (int j = 0; j < n; ++j)
    hipLaunchKernelGGL(k_tridiag_step<NC>, dim3(n / kTriRows, nmat), dim3(256), 0, st, S, j);
  hipLaunchKernelGGL(k_tri_values, dim3((rmax + 3) / 4, nmat), dim3(256), 0, st, S.d, S.e, lam, norm, info, n, rk, rv,
                     rmax);
  const int rt = (rmax + 15) / 16;
  // a matrix whose vectors are orthonormal after a round returns at once from
  // the later ones (4.6 us a launch, 37 us of 8.1 ms for a 32k prompt's first token)
  for (int round = 0; round < kOrthoRounds; ++round) {
    hipLaunchKernelGGL(k_tri_vectors, dim3((rmax + ev - 1) / ev, nmat), dim3(64), 0, st, S.d, S.e, lam, norm, info,
                       state, Z, n, rk, rv, rmax, ev, round);
    hipLaunchKernelGGL(k_z_gram, dim3(rt * (rt + 1) / 2, nmat), dim3(256), 0, st, Z, G, info, state, n, rk, rv, rmax,
                       round);
    hipLaunchKernelGGL(rmax <= kCholLds ? k_z_chol<true> : k_z_chol<false>, dim3(nmat), dim3(1024), 0, st, G, LT, info,
                       state, rk, rv, rmax, round);
    hipLaunchKernelGGL(k_z_solve, dim3(n / 64, nmat), dim3(64), 0, st, Z, G, info, state, n, rk, rv, rmax, round);
  }
  hipLaunchKernelGGL(k_tri_back<NC>, dim3((rmax + 3) / 4, nmat), dim3(256), 0, st, S, Z, rk, rv, rmax);
}
}  // namespace

hipError_t prefill_bases_ws_bytes(const Problem& P, int n_s, size_t* bytes) {
  *bytes = bases_layout(P, n_s).total;
  return hipSuccess;
}

hipError_t launch_prefill_bases(const Problem& P, int64_t n_rows, const void* s_k, const void* s_v, int n_uniform,
                                int n_recent, int center, int32_t* idx_out, void* bases_k, void* bases_v, void* ws,
                                size_t ws_bytes, hipStream_t st) {
  const int n_s = n_uniform + n_recent;
  hipError_t e = hipSuccess;
  const BasesLayout l = bases_layout(P, n_s);
  if (ws_bytes < l.total) return hipErrorInvalidValue;
  char* w = static_cast<char*>(ws);
  auto at = [&](size_t o) { return reinterpret_cast<double*>(w + o); };
  const TriState S{at(l.m), at(l.v), at(l.y), at(l.d), at(l.e), at(l.tau)};
  int32_t* info = reinterpret_cast<int32_t*>(w + l.info);
  int32_t* state = reinterpret_cast<int32_t*>(w + l.state);
  double *inv = at(l.inv), *part = at(l.part), *Z = at(l.z);
  int32_t* idx = reinterpret_cast<int32_t*>(w + l.idx);
  const int nb = P.nb, Dg = P.Dg, Dp = P.Dp, nmat = P.B * 2 * nb;
  const uint16_t* sk = static_cast<const uint16_t*>(s_k);
  const uint16_t* sv = static_cast<const uint16_t*>(s_v);

  hipLaunchKernelGGL(k_sample_hybrid, dim3((n_s + 255) / 256), dim3(256), 0, st, idx, n_rows, n_uniform, n_recent);
  hipLaunchKernelGGL(k_row_norms, dim3((n_s + 3) / 4, 2 * nb, P.B), dim3(256), 0, st, sk, sv, idx, inv, n_rows, n_s,
                     Dp, nb);
  if (center)
    hipLaunchKernelGGL(k_col_partial, dim3(Dg / 256, 2 * nb * kMeanChunks, P.B), dim3(256), 0, st, sk, sv, idx, inv,
                       part, n_rows, n_s, Dp, nb);
  const int nt = Dg / kGramTile;
  hipLaunchKernelGGL(k_gram, dim3(nt * (nt + 1) / 2, 2 * nb, P.B), dim3(256), 0, st, sk, sv, idx, inv, part, S.A,
                     n_rows, n_s, Dp, nb, center);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int rk = P.rank_cfg, rv = P.rank_v_cfg;
#define S4R_EIGEN_CASE(NC) \
  case NC: launch_eigen<NC>(S, at(l.lam), at(l.norm), info, state, Z, at(l.g), at(l.lt), nmat, rk, rv, st); break;
  switch (Dg / 256) {
    S4R_EIGEN_CASE(1)
    S4R_EIGEN_CASE(2)
    S4R_EIGEN_CASE(3)
    S4R_EIGEN_CASE(4)
    S4R_EIGEN_CASE(5)
    S4R_EIGEN_CASE(6)
    S4R_EIGEN_CASE(7)
    S4R_EIGEN_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef S4R_EIGEN_CASE
  const int64_t nel = (int64_t)P.B * nb * Dg * std::max(P.rank, P.rank_v);
  const dim3 grid((unsigned)std::min<int64_t>((nel + 255) / 256, 4096), 2);
  if (P.dtype == S4R_BF16)
    hipLaunchKernelGGL(k_write_bases<uint16_t>, grid, dim3(256), 0, st, Z, info, state, (uint16_t*)bases_k,
                       (uint16_t*)bases_v, P.B, nb, Dg, P.rank, P.rank_v, rk, rv, std::max(rk, rv));
  else
    hipLaunchKernelGGL(k_write_bases<float>, grid, dim3(256), 0, st, Z, info, state, (float*)bases_k, (float*)bases_v, P.B,
                       nb, Dg, P.rank, P.rank_v, rk, rv, std::max(rk, rv));
  if (idx_out) e = hipMemcpyAsync(idx_out, idx, (size_t)n_s * 4, hipMemcpyDeviceToDevice, st);
  if (e == hipSuccess) e = hipGetLastError();
  return e;
}

}  // namespace s4r
