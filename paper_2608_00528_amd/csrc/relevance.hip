// Section 3.2.2 softmax / window mean and the pooling and group-aggregation
// equations of Section 3.2.3 on gfx950: k_relevance turns the stream's exp
// values and statistics into A~ (fp32) and adds to the sequence's radix
// histogram; k_hist_scores builds it for caller-given scores.
#include "s4r_device.h"
#include "s4r_internal.h"
#include "select_key.h"

namespace s4r {

// ---------------------------------------------------------------------------
// K2: relevance A~ and its radix histogram
// ---------------------------------------------------------------------------
// grid (ceil(L / chunk), B), 256 threads; chunk = 1024 / 512 tokens for
// G <= 8 / 16.  The stream's exp values are stored token-major,
// e[b][x][c] for query column c = g * W_q + i (GWP = G * W_q rounded up to a
// multiple of 4, padding columns zero), with one reference per 16-token tile,
// tref[b][tile][c].  Reading the exp values bounds the large batches (8 x 128k
// tokens at 7 columns: 33.5 MB, 8 us at the rate of a large copy), the chain
// of dependent phases the small ones.  One memory latency: the scoring workgroups' statistics,
// the chunk's tile references and its exp values (plus the pooling halo) are
// all requested before any is used.  Then each wave folds query columns'
// statistics into the global (M, S), sums in fp64 (the same fixed order in
// every workgroup, so A~ is deterministic), and the per-tile factors
// exp(ref - M) / S; every exponential there takes its fp64 argument through
// exp_neg_accurate (fp64 range reduction, hardware exp2 of the fraction: about
// one fp32 ulp), far cheaper than an fp64 exp per scoring workgroup and
// column in every workgroup.  Per staged position the window mean
// over the W_q rows is formed once (fp32 products of values exact to about an
// ulp; the max-pooling that follows is exact), staged in LDS, and every thread
// pools consecutive outputs, whose windows overlap (four outputs of a 7-wide
// window read 12 values in three 16-byte reads instead of 28), and sums the
// groups in fp64.  The wave reductions use DPP and lane swaps, the factors one
// thread per (tile, column), and the groups are a loop: unrolled over groups,
// outputs and window widths the kernel was up to 90 KB of code, more than the
// instruction cache, which costs about 0.65 us per KB run through.  Measured
// before and after: 19.2 -> 13.9 us (8 x 128k, 7 columns), 12.5 -> 9.8 (32 x
// 32k, 4), 8.7 -> 6.9 (4 x 128k, 4), 14.6 -> 7.6 (16k, 16 columns of 4 rows),
// 12.2 -> 9.9 (120k windowed).
constexpr int kRelThreads = 256;
// scoring-workgroup statistics per lane that the relevance kernel folds itself
// (KSP, all requested together): 2 (up to 128 scoring workgroups), or 8 (up to
// 512) with one query column per wave: the paper's batch-1 setting at 120k
// has 469, whose separate fold launch cost 4.6 us, while eight per lane cost
// the 128-workgroup shapes 0.5 us.  Beyond that k_fold_stats folds them first.
constexpr int kRelStatPer = 2, kRelStatWide = 8;
template <int NQ>
constexpr int rel_stat_max() {
  return 64 * (NQ == 1 ? kRelStatWide : kRelStatPer);
}

// tokens per workgroup: 1024 (G <= 8) or 512, halved (down to 256) while the
// grid would give fewer than four workgroups per CU.  Measured at 1024, 512
// and 256 tokens: about 1024 workgroups is best at batch 4 (512-token chunks,
// relevance 11.9 -> 10.5 us at 128k), batch 8 and batch 32 (1024-token
// chunks; 512 costs 2.7 and 1 us there).  The histogram copies keep the
// flush atomics of more workgroups from serialising.
constexpr int kRelMinWg = 1024;
// Windows wider than kPoolShared read single values and always take one output
// per thread, so that a wave reads consecutive words: with TPT consecutive
// outputs a thread the reads of neighbouring lanes are TPT words apart and
// conflict (the step over 8 x 128k, 7 columns, with four outputs a thread and one:
// 141 -> 113 us at a window of 33, 191 -> 131 us at 65).
constexpr int kPoolShared = 9;
int relevance_chunk(const Problem& P, int64_t L) {
  if (P.kappa > kPoolShared) return kRelThreads;
  int c = P.G <= 8 ? 1024 : 512;
  while (c > 256 && (int64_t)P.B * ((L + c - 1) / c) < kRelMinWg) c >>= 1;
  return c;
}

// LDS row stride of one group's staged positions (16-byte rows; pool_aggregate
// reads up to 3 values past the window of a chunk's last output)
__host__ __device__ constexpr int rel_row(int span) { return (span + 7) / 4 * 4; }

// Pooling (kappa = 2H + 1, stride 1, same length) and aggregation over the G
// groups for outputs o0 .. o0 + TPT - 1 (o0 a multiple of TPT): the windows of
// neighbouring outputs overlap, so a thread reads TPT + 2H values per group in
// aligned vectors and shares the maximum of the common part.  H < 0 is the
// generic path for wider windows (TPT = 1).
template <int H, int TPT>
__device__ __forceinline__ void pool_aggregate(const float* __restrict__ vs, int row, int o0, int G, int kappa,
                                               int pool_mode, int agg, float (&af)[TPT]) {
  double acc[TPT];
#pragma unroll
  for (int j = 0; j < TPT; ++j) acc[j] = (agg == S4R_AGG_MEAN) ? 0.0 : -INFINITY;
  const bool mean = agg == S4R_AGG_MEAN;
  if constexpr (H >= 0) {
    constexpr int NV = (TPT + 2 * H + TPT - 1) / TPT * TPT;
#pragma unroll 4
    for (int g = 0; g < G; ++g) {
      const float* p = vs + g * row + o0;
      float w[NV];
#pragma unroll
      for (int i = 0; i < NV; i += TPT) {
        if constexpr (TPT == 4)
          *reinterpret_cast<float4*>(&w[i]) = *reinterpret_cast<const float4*>(p + i);
        else if constexpr (TPT == 2)
          *reinterpret_cast<float2*>(&w[i]) = *reinterpret_cast<const float2*>(p + i);
        else
          w[i] = p[i];
      }
      float a[TPT];
      if (pool_mode == S4R_POOL_MAX) {
        if constexpr (2 * H >= TPT - 1) {
          float m = w[TPT - 1];                    // in every output's window
#pragma unroll
          for (int d = TPT; d <= 2 * H; ++d) m = fmaxf(m, w[d]);
#pragma unroll
          for (int j = 0; j < TPT; ++j) {
            float x = m;
#pragma unroll
            for (int d = j; d < TPT - 1; ++d) x = fmaxf(x, w[d]);
#pragma unroll
            for (int d = 2 * H + 1; d <= j + 2 * H; ++d) x = fmaxf(x, w[d]);
            a[j] = x;
          }
        } else {
#pragma unroll
          for (int j = 0; j < TPT; ++j) {
            a[j] = w[j];
#pragma unroll
            for (int d = 1; d <= 2 * H; ++d) a[j] = fmaxf(a[j], w[j + d]);
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < TPT; ++j) {
          double sa = 0.0;
#pragma unroll
          for (int d = 0; d <= 2 * H; ++d) sa += (double)w[j + d];
          a[j] = (float)(sa / kappa);
        }
      }
#pragma unroll
      for (int j = 0; j < TPT; ++j) acc[j] = mean ? acc[j] + (double)a[j] : fmax(acc[j], (double)a[j]);
    }
  } else {
    static_assert(TPT == 1, "one output per thread");
    for (int g = 0; g < G; ++g) {
      const float* v = vs + g * row + o0;
      float a = v[0];
      double sa = (double)v[0];
      for (int d = 1; d < kappa; ++d) {
        a = fmaxf(a, v[d]);
        sa += (double)v[d];
      }
      if (pool_mode != S4R_POOL_MAX) a = (float)(sa / kappa);
      acc[0] = mean ? acc[0] + (double)a : fmax(acc[0], (double)a);
    }
  }
#pragma unroll
  for (int j = 0; j < TPT; ++j) af[j] = (float)(mean ? acc[j] / G : acc[j]);
}

template <int TPT>
__device__ __forceinline__ void pool_dispatch(const float* vs, int row, int o0, int G, int kappa, int pool_mode, int agg,
                                              float (&af)[TPT]) {
  switch (kappa / 2) {
    case 0: pool_aggregate<0, TPT>(vs, row, o0, G, kappa, pool_mode, agg, af); break;
    case 1: pool_aggregate<1, TPT>(vs, row, o0, G, kappa, pool_mode, agg, af); break;
    case 2: pool_aggregate<2, TPT>(vs, row, o0, G, kappa, pool_mode, agg, af); break;
    case 3: pool_aggregate<3, TPT>(vs, row, o0, G, kappa, pool_mode, agg, af); break;
    case kPoolShared / 2: pool_aggregate<kPoolShared / 2, TPT>(vs, row, o0, G, kappa, pool_mode, agg, af); break;
    default:                                               // wider: the launch takes TPT = 1
      if constexpr (TPT == 1) pool_aggregate<-1, TPT>(vs, row, o0, G, kappa, pool_mode, agg, af);
  }
}

// what the kernel's query columns are: one query row per group, several, or
// the newest row of a windowed step
enum RelMode { kRelOne, kRelRows, kRelWindow };

// kRelWindow (windowed step, query window of wrows rows): the stream scored
// only the newest query row (its G columns, Wq = 1 here); the softmax of each
// older row over its own keys comes from the window state
// [B][wrows][G][cap], row slot L_r mod wrows for the row that was newest at
// length L_r (it covers keys < L_r).  This kernel adds the newest row's
// softmax to the older rows' for the window mean and stores it in its slot.
// With a running sum (rsum, longer windows) the older rows' sum per position
// is kept in fp64 as well, in two buffers [2][B][G][cap] by the parity of L:
// the step reads buffer L & 1 and writes buffer (L + 1) & 1 = that sum plus
// the newest row minus the row leaving the window (the one newest at
// L - wrows + 1, masked at its key limit), for the positions it owns.  Without
// one (up to kWinDirectRows rows) the older rows are read directly, four
// positions of a group per unit.  In the 256-token chunks of a small batch
// either is requested with the first loads.
template <int NQ, int TPT, int MODE, int KSP>
__global__ __launch_bounds__(kRelThreads) void k_relevance(
    const float* __restrict__ e, const float* __restrict__ tref, const double* __restrict__ wg_stats,
    const double* __restrict__ col_stats, float* __restrict__ atilde, uint32_t* __restrict__ hist, float* __restrict__ scores_out,
    int64_t cap, int L, int n_hist, int G, int Wq, int kappa, int pool_mode, int agg, int ntiles_cap, int nwg,
    Lens lens, int key_shift, float* __restrict__ state, int wrows, double* __restrict__ rsum, int hist_nc) {
  constexpr int GWP = 4 * NQ;
  constexpr int CHUNK = kRelThreads * TPT;
  constexpr int PPT = TPT + 1;                             // staged positions per thread (span <= CHUNK + 64)
  constexpr int NTL = CHUNK / kTileTok + 6;                // tiles of a chunk and its halo
  constexpr int FPT = (NTL * GWP + kRelThreads - 1) / kRelThreads;
  constexpr bool WIN = MODE == kRelWindow;
  constexpr bool WIN_PRE = WIN && TPT == 1 && NQ == 1;     // older rows with the first loads
  constexpr int UPRE = 2;                                  // units of older rows per thread held ahead
  const int b = blockIdx.y;
  const int score_stride = L;                      // scores_out rows are [B, L] with the call's (largest) L
  {                                                // this sequence's length (ragged batch: n_hist shifts with it)
    const int Lb = (int)len_of(lens, b, L);
    n_hist += Lb - L;
    L = Lb;
  }
  if ((int)blockIdx.x * CHUNK >= L) return;                // past this sequence's end
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int GW = G * Wq;
  const int h = kappa / 2;
  const int t0 = blockIdx.x * CHUNK;
  const int x0 = t0 - h;                                   // first staged position
  const int span = CHUNK + 2 * h;
  const int row = rel_row(span);
  const int tile_lo = max(x0, 0) / kTileTok;
  const int tile_hi = (min(t0 + CHUNK + h, L) - 1) / kTileTok;
  const int nfac = (tile_hi - tile_lo + 1) * GWP;          // <= NTL * GWP

  __shared__ uint32_t hl[kHistBins];
  __shared__ double sM[GWP], sInvS[GWP];
  __shared__ __align__(16) float fac[NTL * GWP];           // exp(ref - M) / S per tile and column
  extern __shared__ __align__(16) float vs[];              // [G][row]: window mean at x0 + i

  // ---- all global reads of this workgroup, issued before any is used ----------
  // statistics: wave w folds columns w, w + 4, .., KSP entries per lane (or,
  // with many scoring workgroups, the global statistics k_fold_stats formed)
  double2 st[NQ][KSP];
  const double2* stats = reinterpret_cast<const double2*>(wg_stats) + (int64_t)b * GW * nwg;
  double2 cs = make_double2(0.0, 0.0);
  if (col_stats) {
    cs = reinterpret_cast<const double2*>(col_stats)[(int64_t)b * GW + min(t, GW - 1)];
  } else {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = min(wave + 4 * q, GW - 1);
#pragma unroll
      for (int k = 0; k < KSP; ++k) st[q][k] = stats[(int64_t)c * nwg + min(lane + 64 * k, nwg - 1)];
    }
  }
  // tile references, contiguous over (tile, column)
  float rf[FPT];
  {
    const float* tp = tref + ((int64_t)b * ntiles_cap + tile_lo) * GWP;
#pragma unroll
    for (int k = 0; k < FPT; ++k) rf[k] = tp[min(t + k * kRelThreads, nfac - 1)];
  }
  // exp values of the staged positions (clamped into the span and [0, L); masked later)
  float4 ev[PPT][NQ];
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const int x = min(max(x0 + min(t + k * kRelThreads, span - 1), 0), L - 1);
    const float4* ep = reinterpret_cast<const float4*>(e + ((int64_t)b * cap + x) * GWP);
#pragma unroll
    for (int q = 0; q < NQ; ++q) ev[k][q] = ep[q];
  }
  // the window state: running sum and leaving row per staged position, or
  // units of older rows
  float* sb = WIN ? state + (int64_t)b * wrows * G * cap : nullptr;
  const double* scur = nullptr;
  double* snext = nullptr;
  const float* sold = nullptr;
  const int Lo = L - wrows + 1;                            // the leaving row was newest at Lo
  double so[WIN_PRE ? PPT : 1][GWP];
  float po[WIN_PRE ? PPT : 1][GWP];
  const int u0 = (x0 >= 0 ? x0 : x0 - 3) / 4;              // floor(x0 / 4)
  const int nu = (x0 + span + 3) / 4 - u0;                 // units covering the staged positions
  float4 old[WIN_PRE ? UPRE : 1][kWinDirectRows - 1];
  // the older rows (ages 1 .. wrows - 1, slot (L - a) mod wrows) of unit w
  auto load_unit = [&](int w, float4 (&o)[kWinDirectRows - 1]) __attribute__((always_inline)) {
    const int g = w / nu;
    const int xl = min(max(4 * (u0 + w % nu), 0), (int)(cap - 4));
#pragma unroll
    for (int v = 0; v < kWinDirectRows - 1; ++v) {
      const int a = min(1 + v, wrows - 1);
      const int slot = ((L - a) % wrows + wrows) % wrows;  // L - a < 0 early on: masked
      o[v] = *reinterpret_cast<const float4*>(sb + ((int64_t)slot * G + g) * cap + xl);
    }
  };
  if constexpr (WIN) {
    if (rsum) {
      scur = rsum + ((int64_t)(L & 1) * gridDim.y + b) * G * cap;
      snext = rsum + ((int64_t)((L + 1) & 1) * gridDim.y + b) * G * cap;
      sold = sb + (int64_t)((Lo % wrows + wrows) % wrows) * G * cap;
    }
    if constexpr (WIN_PRE) {
      if (rsum) {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
          const int x = min(max(x0 + min(t + k * kRelThreads, span - 1), 0), (int)cap - 1);
#pragma unroll
          for (int c = 0; c < GWP; ++c) {
            so[k][c] = scur[(int64_t)min(c, G - 1) * cap + x];
            po[k][c] = sold[(int64_t)min(c, G - 1) * cap + x];
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < UPRE; ++i) load_unit(min(t + i * kRelThreads, G * nu - 1), old[i]);
      }
    }
  }
  for (int i = t; i < kHistBins; i += kRelThreads) hl[i] = 0;

  // ---- global (M, S) of each query column ---------------------------------------------
  if (col_stats) {
    if (t < GW) {
      sM[t] = cs.x;
      sInvS[t] = cs.y;
    }
  } else {                                                 // nwg <= 64 * KSP
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = wave + 4 * q;
      if (c < GW) {                                        // wave-uniform
        float m = -INFINITY;                               // maxima are fp32 values
#pragma unroll
        for (int k = 0; k < KSP; ++k) m = fmaxf(m, lane + 64 * k < nwg ? (float)st[q][k].x : -INFINITY);
        m = wave_max(m);
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < KSP; ++k) {
          const bool live = lane + 64 * k < nwg && st[q][k].x != -INFINITY;
          const double x = st[q][k].y * (double)exp_neg_accurate(live ? st[q][k].x - (double)m : 0.0);
          s += live ? x : 0.0;
        }
        s = wave_sum(s);
        if (lane == 0) {
          sM[c] = (double)m;
          sInvS[c] = 1.0 / s;
        }
      }
    }
  }
  __syncthreads();
  // ---- per-tile factors ---------------------------------------------------------------
#pragma unroll
  for (int k = 0; k < FPT; ++k) {
    const int i = t + k * kRelThreads, c = i % GWP;
    if (i < nfac)
      fac[i] = (c < GW && rf[k] != -INFINITY)
                   ? (float)((double)exp_neg_accurate((double)rf[k] - sM[c]) * sInvS[c]) : 0.f;
  }
  __syncthreads();
  // ---- window mean over the W_q rows of every staged position -------------------------
  const float pad = (pool_mode == S4R_POOL_MAX) ? -INFINITY : 0.f;
  const float inv_wq = 1.f / (float)(WIN ? wrows : Wq);
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const int i = t + k * kRelThreads;
    if (i < span) {
      const int x = x0 + i;
      const bool in = x >= 0 && x < L;
      const float* fr = fac + (min(max(x, 0), L - 1) / kTileTok - tile_lo) * GWP;
      float ex[GWP];                                       // the probabilities
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const float4 f4 = *reinterpret_cast<const float4*>(fr + 4 * q);
        ex[4 * q] = ev[k][q].x * f4.x;
        ex[4 * q + 1] = ev[k][q].y * f4.y;
        ex[4 * q + 2] = ev[k][q].z * f4.z;
        ex[4 * q + 3] = ev[k][q].w * f4.w;
      }
      if constexpr (WIN) {
        // the newest row's softmax: into its slot (own chunk) and into LDS;
        // the older rows are added from the running sum, else below
        const bool own = in && x >= t0 && x < t0 + CHUNK;
        float* snew = sb + (int64_t)(L % wrows) * G * cap;
        const int xc = min(max(x, 0), (int)cap - 1);
#pragma unroll
        for (int c = 0; c < GWP; ++c) {
          if (c < G) {
            const float pn = in ? ex[c] : 0.f;
            if (own) snew[(int64_t)c * cap + x] = pn;
            float v = pn;
            if (rsum) {
              const double s0 = WIN_PRE ? so[WIN_PRE ? k : 0][c] : scur[(int64_t)c * cap + xc];
              const float p0 = WIN_PRE ? po[WIN_PRE ? k : 0][c] : sold[(int64_t)c * cap + xc];
              const double sn = s0 + (double)pn;
              if (own) snext[(int64_t)c * cap + x] = sn - (x < Lo ? (double)p0 : 0.0);
              v = in ? (float)(sn * (double)inv_wq) : pad;
            }
            vs[c * row + i] = v;
          }
        }
      } else if constexpr (MODE == kRelOne) {
#pragma unroll
        for (int c = 0; c < GWP; ++c)
          if (c < G) vs[c * row + i] = in ? ex[c] : pad;
      } else {
        // columns g * Wq .. (g + 1) * Wq - 1 are group g's rows
        float sum = 0.f;
        int left = Wq, g = 0;                              // uniform
#pragma unroll
        for (int c = 0; c < GWP; ++c) {
          if (g < G) {
            sum += ex[c];
            if (--left == 0) {
              vs[g * row + i] = in ? sum * inv_wq : pad;
              sum = 0.f;
              left = Wq;
              ++g;
            }
          }
        }
      }
    }
  }
  __syncthreads();
  if constexpr (WIN) {
    if (!rsum) {                                           // (uniform: a kernel argument)
      // older rows: the row of age a covers keys < L - a
      auto add_unit = [&](int w, const float4 (&o)[kWinDirectRows - 1]) __attribute__((always_inline)) {
        const int g = w / nu, xu = 4 * (u0 + w % nu);      // first position of the unit
        const int xl = min(max(xu, 0), (int)(cap - 4));
        float sv[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < kWinDirectRows - 1; ++v) {
          const int lim = 1 + v < wrows ? L - (1 + v) : 0;   // keys of this row
          const float o4[4] = {o[v].x, o[v].y, o[v].z, o[v].w};
#pragma unroll
          for (int j = 0; j < 4; ++j) sv[j] += xl + j < lim ? o4[j] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int x = xu + j, i = x - x0;
          if (i >= 0 && i < span) {
            const bool in = x >= 0 && x < L && xl == xu;
            vs[g * row + i] = in ? (vs[g * row + i] + sv[j]) * inv_wq : pad;
          }
        }
      };
      int w = t;
      if constexpr (WIN_PRE) {
#pragma unroll
        for (int i = 0; i < UPRE; ++i, w += kRelThreads)
          if (w < G * nu) add_unit(w, old[i]);
      }
      for (; w < G * nu; w += kRelThreads) {
        float4 o[kWinDirectRows - 1];
        load_unit(w, o);
        add_unit(w, o);
      }
      __syncthreads();
    }
  }
  // ---- pooling (kappa, stride 1, same length) and aggregation over G -------------------
  float af[TPT];
  pool_dispatch<TPT>(vs, row, t * TPT, G, kappa, pool_mode, agg, af);
  const int xo = t0 + t * TPT;
  float* ap = atilde + (int64_t)b * cap + xo;              // cap is a multiple of 16: aligned for TPT values
  if constexpr (TPT == 4) {
    if (xo + 3 < L) *reinterpret_cast<float4*>(ap) = make_float4(af[0], af[1], af[2], af[3]);
  } else if constexpr (TPT == 2) {
    if (xo + 1 < L) *reinterpret_cast<float2*>(ap) = make_float2(af[0], af[1]);
  }
#pragma unroll
  for (int j = 0; j < TPT; ++j) {
    const int x = xo + j;
    if (x < L) {
      if (TPT == 1 || xo + TPT > L) ap[j] = af[j];
      if (scores_out) scores_out[(int64_t)b * score_stride + x] = af[j];
    }
    if (x < n_hist) atomicAdd(&hl[selection_key_shift(af[j], key_shift) >> kHistShift], 1u);
  }
  __syncthreads();
  // this workgroup's histogram into the sequence's (zeroed by the query
  // projection earlier in the step): one global atomic per non-empty bin
  uint32_t* hs = hist + (int64_t)b * kHistStride + (blockIdx.x & (hist_nc - 1)) * kHistBins;
  for (int i = t; i < kHistBins; i += kRelThreads) {
    const uint32_t c = hl[i];
    if (c) atomicAdd(&hs[i], c);
  }
}

// K2 for more than 16 query columns (G * W_q up to 128, the paper's tied
// W_q = W = 32): grid (ceil(L / 256), B), 256 threads, 256 tokens per
// workgroup.  The global (M, 1 / S) of every column comes from k_fold_stats;
// the per-tile factors exp(ref - M) / S of the chunk's tiles (and halo) go to
// LDS; thread (position, group) forms the window mean of its group's W_q
// columns from the exp values (contiguous per position) with an fp64 sum of
// the fp32 products, then pooling and group aggregation run as in k_relevance.
constexpr int kWideChunk = kRelThreads;
constexpr int kWideMaxTiles = (kWideChunk + 64) / kTileTok + 2;

__global__ __launch_bounds__(kRelThreads) void k_relevance_wide(
    const float* __restrict__ e, const float* __restrict__ tref, const double* __restrict__ col_stats,
    float* __restrict__ atilde, uint32_t* __restrict__ hist, float* __restrict__ scores_out, int64_t cap, int L,
    int n_hist, int G, int Wq, int gwp, int kappa, int pool_mode, int agg, int ntiles_cap, Lens lens, int key_shift,
    int hist_nc) {
  const int b = blockIdx.y;
  const int score_stride = L;
  {
    const int Lb = (int)len_of(lens, b, L);
    n_hist += Lb - L;
    L = Lb;
  }
  if ((int)blockIdx.x * kWideChunk >= L) return;
  const int t = threadIdx.x;
  const int GW = G * Wq;
  const int h = kappa / 2;
  const int t0 = blockIdx.x * kWideChunk;
  const int x0 = t0 - h;
  const int span = kWideChunk + 2 * h;
  const int row = rel_row(span);
  const int tile_lo = max(x0, 0) / kTileTok;
  const int tile_hi = (min(t0 + kWideChunk + h, L) - 1) / kTileTok;
  const int ntl = tile_hi - tile_lo + 1;                   // <= kWideMaxTiles

  __shared__ uint32_t hl[kHistBins];
  __shared__ __align__(16) float fac[kWideMaxTiles * kMaxGW];   // [tile][column]
  extern __shared__ __align__(16) float vs[];              // [G][row]
  for (int i = t; i < kHistBins; i += kRelThreads) hl[i] = 0;
  const double2* cs = reinterpret_cast<const double2*>(col_stats) + (int64_t)b * GW;
  for (int i = t; i < ntl * GW; i += kRelThreads) {
    const int tl = i / GW, c = i % GW;
    const float r = tref[((int64_t)b * ntiles_cap + tile_lo + tl) * gwp + c];
    const double2 st = cs[c];
    fac[tl * GW + c] = (r != -INFINITY) ? (float)((double)exp_neg_accurate((double)r - st.x) * st.y) : 0.f;
  }
  __syncthreads();
  // window mean over the W_q rows of group g at every staged position
  const float pad = (pool_mode == S4R_POOL_MAX) ? -INFINITY : 0.f;
  const double inv_wq = 1.0 / (double)Wq;
  for (int i = t; i < span * G; i += kRelThreads) {
    const int xi = i / G, g = i % G;
    const int x = x0 + xi;
    float v = pad;
    if (x >= 0 && x < L) {
      const float* ep = e + ((int64_t)b * cap + x) * gwp + g * Wq;
      const float* fr = fac + (x / kTileTok - tile_lo) * GW + g * Wq;
      double sum = 0.0;                            // W_q products summed in fp64
      if ((Wq & 3) == 0) {                         // 16-byte loads (rows of gwp, a multiple of 16, floats)
        const float4* e4 = reinterpret_cast<const float4*>(ep);
        const float4* f4 = reinterpret_cast<const float4*>(fr);
        for (int c = 0; c < Wq / 4; ++c) {
          const float4 a = e4[c], f = f4[c];
          sum += (double)a.x * (double)f.x + (double)a.y * (double)f.y + (double)a.z * (double)f.z +
                 (double)a.w * (double)f.w;
        }
      } else {
        for (int c = 0; c < Wq; ++c) sum += (double)ep[c] * (double)fr[c];
      }
      v = (float)(sum * inv_wq);
    }
    vs[g * row + xi] = v;
  }
  __syncthreads();
  float af[1];
  pool_dispatch<1>(vs, row, t, G, kappa, pool_mode, agg, af);
  const int x = t0 + t;
  if (x < L) {
    atilde[(int64_t)b * cap + x] = af[0];
    if (scores_out) scores_out[(int64_t)b * score_stride + x] = af[0];
  }
  if (x < n_hist) atomicAdd(&hl[selection_key_shift(af[0], key_shift) >> kHistShift], 1u);
  __syncthreads();
  uint32_t* hs = hist + (int64_t)b * kHistStride + (blockIdx.x & (hist_nc - 1)) * kHistBins;
  for (int i = t; i < kHistBins; i += kRelThreads) {
    const uint32_t c = hl[i];
    if (c) atomicAdd(&hs[i], c);
  }
}

// histogram of caller-provided scores (standalone selection), into a
// histogram zeroed by k_zero_hist
__global__ __launch_bounds__(256) void k_zero_hist(uint32_t* __restrict__ hist, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) hist[i] = 0u;
}

__global__ __launch_bounds__(256) void k_hist_scores(const float* __restrict__ scores, uint32_t* __restrict__ hist,
                                                     int L, int n_hist, int hist_nc) {
  const int b = blockIdx.y;
  __shared__ uint32_t hl[kHistBins];
  for (int i = threadIdx.x; i < kHistBins; i += blockDim.x) hl[i] = 0;
  __syncthreads();
  const int t0 = blockIdx.x * kHistChunk;
  for (int i = threadIdx.x; i < kHistChunk; i += blockDim.x) {
    const int x = t0 + i;
    if (x < n_hist) atomicAdd(&hl[selection_key(scores[(int64_t)b * L + x]) >> kHistShift], 1u);
  }
  __syncthreads();
  uint32_t* hs = hist + (int64_t)b * kHistStride + (blockIdx.x & (hist_nc - 1)) * kHistBins;
  for (int i = threadIdx.x; i < kHistBins; i += blockDim.x) {
    const uint32_t c = hl[i];
    if (c) atomicAdd(&hs[i], c);
  }
}

// Global (max, 1 / sum) of every query column's softmax over the length,
// folded once from the scoring workgroups' (max, sum) pairs when there are
// more than the relevance kernel folds itself (rel_stat_max): grid (GW,
// B), thread t folds pairs t, t + 256, ... in order, then a fixed-order tree
// across the threads (deterministic).
__global__ __launch_bounds__(256) void k_fold_stats(const double* __restrict__ wg_stats, double* __restrict__ col_stats,
                                                    int GW, int nwg) {
  const int c = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
  const double2* row = reinterpret_cast<const double2*>(wg_stats) + ((int64_t)b * GW + c) * nwg;
  __shared__ double sm[256], ss[256];
  auto merge = [](double& M, double& S, double m, double s) {
    if (m == -INFINITY) return;
    const double Mn = fmax(M, m);
    S = ((M == -INFINITY) ? 0.0 : S * (double)exp_neg_accurate(M - Mn)) + s * (double)exp_neg_accurate(m - Mn);
    M = Mn;
  };
  double M = -INFINITY, S = 0.0;
  for (int w0 = 0; w0 < nwg; w0 += 4 * 256) {
    double2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = row[min(w0 + k * 256 + t, nwg - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (w0 + k * 256 + t < nwg) merge(M, S, v[k].x, v[k].y);
  }
  sm[t] = M;
  ss[t] = S;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) {
      double M2 = sm[t], S2 = ss[t];
      merge(M2, S2, sm[t + o], ss[t + o]);
      sm[t] = M2;
      ss[t] = S2;
    }
    __syncthreads();
  }
  if (t == 0) reinterpret_cast<double2*>(col_stats)[(int64_t)b * GW + c] = make_double2(sm[0], 1.0 / ss[0]);
}

template <int NQ, int TPT>
static void launch_rel_t(const Problem& P, const Workspace& ws, int64_t L, float* scores_out, hipStream_t st) {
  const int n_hist = (int)std::max<int64_t>(L - P.W, 0);
  constexpr int chunk = kRelThreads * TPT;
  const size_t lds = (size_t)P.G * rel_row(chunk + 2 * (P.kappa / 2)) * sizeof(float);
  dim3 grid((unsigned)((L + chunk - 1) / chunk), P.B);
  const int nwg = score_workgroups(P, L);
  const bool fold = nwg > rel_stat_max<NQ>();
  constexpr int KW = NQ == 1 ? kRelStatWide : kRelStatPer;   // (only one column per wave folds 512)
  auto kern = nwg > 64 * kRelStatPer && !fold
                  ? (P.Wq == 1 ? k_relevance<NQ, TPT, kRelOne, KW> : k_relevance<NQ, TPT, kRelRows, KW>)
                  : (P.Wq == 1 ? k_relevance<NQ, TPT, kRelOne, kRelStatPer>
                               : k_relevance<NQ, TPT, kRelRows, kRelStatPer>);
  if (fold) hipLaunchKernelGGL(k_fold_stats, dim3(P.GW, P.B), dim3(256), 0, st, ws.wg_stats, ws.col_stats, P.GW, nwg);
  hipLaunchKernelGGL(kern, grid, dim3(kRelThreads), lds, st, ws.e, ws.run_m, ws.wg_stats,
                     fold ? ws.col_stats : nullptr, ws.atilde, ws.hist, scores_out, P.cap, (int)L, n_hist, P.G, P.Wq, P.kappa, P.pool_mode, P.agg,
                     (int)(P.cap / kTileTok), nwg, P.lens, fused_key_shift(P, L), nullptr, 1, nullptr,
                     hist_copies(grid.x));
}

template <int NQ>
static void launch_rel_nq(const Problem& P, const Workspace& ws, int64_t L, float* scores_out, hipStream_t st) {
  switch (relevance_chunk(P, L)) {
    case 1024: launch_rel_t<NQ, 4>(P, ws, L, scores_out, st); break;
    case 512: launch_rel_t<NQ, 2>(P, ws, L, scores_out, st); break;
    default: launch_rel_t<NQ, 1>(P, ws, L, scores_out, st); break;
  }
}

// more than 16 query columns: the statistics are always folded first
static void launch_rel_wide(const Problem& P, const Workspace& ws, int64_t L, float* scores_out, hipStream_t st) {
  const int n_hist = (int)std::max<int64_t>(L - P.W, 0);
  const int nwg = score_workgroups(P, L);
  hipLaunchKernelGGL(k_fold_stats, dim3(P.GW, P.B), dim3(256), 0, st, ws.wg_stats, ws.col_stats, P.GW, nwg);
  const size_t lds = (size_t)P.G * rel_row(kWideChunk + 2 * (P.kappa / 2)) * sizeof(float);
  dim3 grid((unsigned)((L + kWideChunk - 1) / kWideChunk), P.B);
  hipLaunchKernelGGL(k_relevance_wide, grid, dim3(kRelThreads), lds, st, ws.e, ws.run_m, ws.col_stats, ws.atilde, ws.hist,
                     scores_out, P.cap, (int)L, n_hist, P.G, P.Wq, gw_padded(P), P.kappa, P.pool_mode, P.agg,
                     (int)(P.cap / kTileTok), P.lens, fused_key_shift(P, L), hist_copies(grid.x));
}

hipError_t launch_relevance(const Problem& P, const Workspace& ws, int64_t L, float* scores_out, hipStream_t st) {
  if (P.GW > kColBlk) {
    launch_rel_wide(P, ws, L, scores_out, st);
    return hipGetLastError();
  }
  switch (gw_padded(P) / 4) {
    case 1: launch_rel_nq<1>(P, ws, L, scores_out, st); break;
    case 2: launch_rel_nq<2>(P, ws, L, scores_out, st); break;
    case 3: launch_rel_nq<3>(P, ws, L, scores_out, st); break;
    default: launch_rel_nq<4>(P, ws, L, scores_out, st); break;
  }
  return hipGetLastError();
}

template <int NQ, int TPT>
static void launch_rel_win_t(const Problem& P1, const Workspace& ws, int64_t L, float* scores_out, float* state,
                             int wrows, hipStream_t st) {
  const int n_hist = (int)std::max<int64_t>(L - P1.W, 0);
  constexpr int chunk = kRelThreads * TPT;
  const size_t lds = (size_t)P1.G * rel_row(chunk + 2 * (P1.kappa / 2)) * sizeof(float);
  dim3 grid((unsigned)((L + chunk - 1) / chunk), P1.B);
  const int nwg = score_workgroups(P1, L);
  const bool fold = nwg > rel_stat_max<NQ>();
  if (fold) hipLaunchKernelGGL(k_fold_stats, dim3(P1.GW, P1.B), dim3(256), 0, st, ws.wg_stats, ws.col_stats, P1.GW, nwg);
  constexpr int KW = NQ == 1 ? kRelStatWide : kRelStatPer;
  auto kern = nwg > 64 * kRelStatPer && !fold ? k_relevance<NQ, TPT, kRelWindow, KW>
                                              : k_relevance<NQ, TPT, kRelWindow, kRelStatPer>;
  hipLaunchKernelGGL(kern, grid, dim3(kRelThreads), lds, st, ws.e, ws.run_m, ws.wg_stats,
                     fold ? ws.col_stats : nullptr, ws.atilde, ws.hist, scores_out, P1.cap, (int)L, n_hist, P1.G, 1,
                     P1.kappa, P1.pool_mode, P1.agg, (int)(P1.cap / kTileTok), nwg, P1.lens, fused_key_shift(P1, L),
                     state, wrows, window_rsum(P1, state, wrows), hist_copies(grid.x));
}

int relevance_hist_copies(const Problem& P, int64_t L, int wrows) {
  const int chunk = (wrows < 2 && P.GW > kColBlk) ? kWideChunk : relevance_chunk(P, L);
  return hist_copies((L + chunk - 1) / chunk);
}

template <int NQ>
static void launch_rel_win_nq(const Problem& P1, const Workspace& ws, int64_t L, float* scores_out, float* state,
                              int wrows, hipStream_t st) {
  switch (relevance_chunk(P1, L)) {
    case 1024: launch_rel_win_t<NQ, 4>(P1, ws, L, scores_out, state, wrows, st); break;
    case 512: launch_rel_win_t<NQ, 2>(P1, ws, L, scores_out, state, wrows, st); break;
    default: launch_rel_win_t<NQ, 1>(P1, ws, L, scores_out, state, wrows, st); break;
  }
}

hipError_t launch_relevance_windowed(const Problem& P1, const Workspace& ws, int64_t L, float* scores_out,
                                     float* state, int wrows, hipStream_t st) {
  switch (gw_padded(P1) / 4) {
    case 1: launch_rel_win_nq<1>(P1, ws, L, scores_out, state, wrows, st); break;
    case 2: launch_rel_win_nq<2>(P1, ws, L, scores_out, state, wrows, st); break;
    case 3: launch_rel_win_nq<3>(P1, ws, L, scores_out, state, wrows, st); break;
    default: launch_rel_win_nq<4>(P1, ws, L, scores_out, state, wrows, st); break;
  }
  return hipGetLastError();
}

// window state of the W_q - 1 older rows from a stream over them (P0: those
// rows as the query window, scored to length L - 1): row r < wrows - 1 covers
// keys < L_r = L - (wrows - 1 - r) and goes to slot L_r mod wrows.  grid
// (ceil(cap / 256), B); the softmax probability of (row, group, key) is its
// exp value times exp(ref - M) / S of its tile and column (fp64 argument, as
// in the relevance kernel).  With a running sum, buffer L & 1 gets the older
// rows' fp64 sum (oldest row first; 0 where no row covers the key) and buffer
// (L + 1) & 1 zeros, over the whole capacity.
__global__ __launch_bounds__(256) void k_window_store(const float* __restrict__ e, const float* __restrict__ tref,
                                                      const double* __restrict__ col_stats, float* __restrict__ state,
                                                      double* __restrict__ rsum, int64_t cap, int L, int G, int wrows,
                                                      int gwp, int ntiles_cap) {
  const int b = blockIdx.y, x = blockIdx.x * 256 + threadIdx.x;
  const int w0 = wrows - 1;                       // rows in the stream, column c = g * w0 + r
  if (x >= cap) return;
  for (int g = 0; g < G; ++g) {
    double sum = 0.0;
    for (int r = 0; r < w0; ++r) {
      const int Lr = L - (w0 - r);
      if (x >= Lr) continue;
      const int c = g * w0 + r;
      const double2 cs = reinterpret_cast<const double2*>(col_stats)[(int64_t)b * G * w0 + c];
      const float ref = tref[((int64_t)b * ntiles_cap + x / kTileTok) * gwp + c];
      const float fac = (ref != -INFINITY) ? (float)((double)exp_neg_accurate((double)ref - cs.x) * cs.y) : 0.f;
      const float p = e[((int64_t)b * cap + x) * gwp + c] * fac;
      state[(((int64_t)b * wrows + Lr % wrows) * G + g) * cap + x] = p;
      sum += (double)p;
    }
    if (rsum) {
      rsum[(((int64_t)(L & 1) * gridDim.y + b) * G + g) * cap + x] = sum;
      rsum[(((int64_t)((L + 1) & 1) * gridDim.y + b) * G + g) * cap + x] = 0.0;
    }
  }
}

hipError_t launch_window_store(const Problem& P0, const Workspace& ws, int64_t L, float* state, int wrows,
                               hipStream_t st) {
  const int nwg = score_workgroups(P0, L - 1);
  hipLaunchKernelGGL(k_fold_stats, dim3(P0.GW, P0.B), dim3(256), 0, st, ws.wg_stats, ws.col_stats, P0.GW, nwg);
  hipLaunchKernelGGL(k_window_store, dim3((unsigned)((P0.cap + 255) / 256), P0.B), dim3(256), 0, st, ws.e,
                     ws.run_m, ws.col_stats, state, window_rsum(P0, state, wrows), P0.cap, (int)L, P0.G, wrows,
                     gw_padded(P0), (int)(P0.cap / kTileTok));
  return hipGetLastError();
}

hipError_t launch_hist_only(const Problem& P, const Workspace& ws, int64_t L, const float* scores, hipStream_t st) {
  const int n_hist = (int)std::max<int64_t>(L - P.W, 0);
  const int ng = std::max(1, (n_hist + kHistChunk - 1) / kHistChunk);
  hipLaunchKernelGGL(k_zero_hist, dim3((P.B * kHistStride + 255) / 256), dim3(256), 0, st, ws.hist,
                     P.B * kHistStride);
  hipLaunchKernelGGL(k_hist_scores, dim3(ng, P.B), dim3(256), 0, st, scores, ws.hist, (int)L, n_hist,
                     hist_copies(ng));
  return hipGetLastError();
}

}  // namespace s4r
