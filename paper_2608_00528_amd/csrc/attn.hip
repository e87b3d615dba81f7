// Sparse reconstruction and final attention of Section 3.2.3 on gfx950.
//
//   k_attn_split  one workgroup per (split, kv head j, sequence).  Wave w owns
//                 the dimension pair blocks {w, w + d_h/32} of head j (16 dims
//                 each, so every RoPE pair (i, i + d_h/2) sits in one lane).
//                 Per 16-token tile of the index list it gathers the selected
//                 coefficient rows (64-byte pieces of the tiled cache) as MFMA
//                 B operands and forms K^T = B^K_j C^T and V^T = B^V_j C^T with
//                 bf16 MFMA (basis rows as A operands: the key basis staged in LDS,
//                 the value basis in registers), so a
//                 lane ends with 8 dims of one token.  RoPE is applied to the
//                 fp32 accumulators, partial logits are summed over the lane's
//                 k-group and across the waves through LDS, and each lane runs
//                 an online softmax for its token slot.  Reconstructed K/V never
//                 leave registers.  The split's (max, sum, output) is written
//                 once after merging the 16 token slots.
//   k_attn_combine one workgroup per (query head, sequence): sink tokens and
//                 the optional exact window KV (full precision, fp32 VALU) and
//                 the merge of all splits into O_t.
//   k_reconstruct / k_sparse_attn: the separately callable reconstruction
//                 (fp32 K^, V^ written out) and attention over given rows.
#include "attn_common.h"

namespace s4r {

// ---------------------------------------------------------------------------
// combine: sinks, exact window, splits -> O_t
// ---------------------------------------------------------------------------
// One workgroup per (query head, sequence).  Every split's (max, sum, output)
// is requested up front (thread t holds float4 t, t + 256, ... of the splits'
// outputs, i.e. dims 4 t % d_h .. + 3 of several splits), together with the key and value rows
// of the first kPreTok extra full-precision tokens (the sinks; further rows
// of an optional exact window are loaded as they are reached).  The extra
// tokens are attended on the VALU with the same fixed-point RoPE phases, and
// the partials are merged with the usual max rescaling.
constexpr int kMaxExtra = 1024 + 64;   // sinks + exact window rows
constexpr int kCombVec = kMaxSplit * 128 / (4 * 256);   // float4 of split outputs per thread
constexpr int kPreTok = 4;             // extra tokens whose rows come with the first loads

// CV: float4 of split outputs per thread, the smallest of 1, 2, 4, kCombVec
// that covers nsplit * d_h / 4 (the launch picks it)
template <typename T, int CV>
__global__ __launch_bounds__(256) void k_attn_combine(
    const T* __restrict__ q, const T* __restrict__ sink_k, const T* __restrict__ sink_v,
    const T* __restrict__ win_k, const T* __restrict__ win_v, const float* __restrict__ part_ml,
    const float* __restrict__ part_o, float* __restrict__ out, int nsplit, int hq, int hkv, int dh,
    int s_sink, int W, int64_t L, double rope_ratio, Lens lens) {
  const int h = blockIdx.x, b = blockIdx.y;
  L = len_of(lens, b, L);
  const int G = hq / hkv, j = h / G;
  const int Dp = hkv * dh;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t pos_q = s_sink + L - 1;
  const int n_win = win_k ? (int)min<int64_t>(W, L) : 0;
  const int n_extra = s_sink + n_win;
  const int half = dh / 2;
  const int64_t pb = ((int64_t)b * hq + h) * kMaxSplit;
  const float sqrt_d = sqrtf((float)dh);

  __shared__ float qr[128];
  __shared__ uint64_t fq[64];
  __shared__ float lg[kMaxExtra];
  __shared__ float s_as[kMaxSplit];
  __shared__ float red[1024];
  __shared__ float s_me, s_den, s_ae;

  // ---- every load of the split partials and the query, issued together -----------------
  const int ne4 = nsplit * dh / 4;                // float4 of split outputs (d_h is a multiple of 4)
  const int ldh = __builtin_ctz(dh);               // head_dim is a power of two
  float4 po[CV];
  const float4* po4 = reinterpret_cast<const float4*>(part_o + pb * dh);
#pragma unroll
  for (int i = 0; i < CV; ++i) po[i] = po4[max(min(t + 256 * i, ne4 - 1), 0)];   // masked below
  float2 ml = make_float2(-INFINITY, 0.f);
  if (t < nsplit) ml = reinterpret_cast<const float2*>(part_ml)[pb + t];
  float xl = 0.f, xh = 0.f;
  if (t < half) {
    const int64_t qo = ((int64_t)b * hq + h) * dh;
    xl = load_elem(q, qo + t);
    xh = load_elem(q, qo + t + half);
  }
  auto krow = [&](int e) -> const T* {
    if (e < s_sink) return sink_k + ((int64_t)b * s_sink + e) * Dp + (int64_t)j * dh;
    return win_k + ((int64_t)b * W + (W - n_win) + (e - s_sink)) * Dp + (int64_t)j * dh;
  };
  auto vrow = [&](int e) -> const T* {
    if (e < s_sink) return sink_v + ((int64_t)b * s_sink + e) * Dp + (int64_t)j * dh;
    return win_v + ((int64_t)b * W + (W - n_win) + (e - s_sink)) * Dp + (int64_t)j * dh;
  };
  auto kpos = [&](int e) -> int64_t { return e < s_sink ? (int64_t)e : (int64_t)s_sink + (L - n_win) + (e - s_sink); };
  // key row of extra token `wave` (lane = RoPE pair) and value rows of the
  // first kPreTok extra tokens (thread t < d_h = dim t)
  float pkl = 0.f, pkh = 0.f;
  if (wave < n_extra && lane < half) {
    const T* kp = krow(wave);
    pkl = load_elem(kp, lane);
    pkh = load_elem(kp, lane + half);
  }
  float pv[kPreTok];
#pragma unroll
  for (int e = 0; e < kPreTok; ++e) pv[e] = (e < n_extra && t < dh) ? load_elem(vrow(e), t) : 0.f;

  // ---- rotated query ----------------------------------------------------------------------
  if (t < half) {
    uint64_t F[4];
    rope_freqs_fixed(rope_ratio, t, F);
    fq[t] = F[0];
    float c, sn;
    rope_cs_fixed(pos_q, F[0], c, sn);
    qr[t] = xl * c - xh * sn;
    qr[t + half] = xh * c + xl * sn;
  }
  __syncthreads();
  // ---- logits of the full-precision tokens: one wave per token, lane = RoPE pair ---------
  for (int e = wave; e < n_extra; e += 4) {
    float part = 0.f;
    if (lane < half) {
      const T* kp = krow(e);
      const float kl = (e == wave) ? pkl : load_elem(kp, lane), kh = (e == wave) ? pkh : load_elem(kp, lane + half);
      float c, sn;
      rope_cs_fixed(kpos(e), fq[lane], c, sn);
      part = qr[lane] * (kl * c - kh * sn) + qr[lane + half] * (kh * c + kl * sn);
    }
    part = wave_sum(part);
    if (lane == 0) lg[e] = part / sqrt_d;
  }
  __syncthreads();
  // ---- (max, sum) of the extra tokens, global maximum, split weights (wave 0) ------------
  if (wave == 0) {
    // (finite also where every logit is -inf: such tokens weigh 0 beside others)
    float mx = -__FLT_MAX__;
    for (int e = lane; e < n_extra; e += 64) mx = fmaxf(mx, lg[e]);
    mx = wave_max(mx);
    float sm = 0.f;
    for (int e = lane; e < n_extra; e += 64) sm += __expf(lg[e] - mx);
    sm = wave_sum(sm);
    const float ms = (lane < nsplit) ? ml.x : -INFINITY;
    const float M = fmaxf(mx, wave_max(ms));
    const float ae = (n_extra > 0) ? __expf(mx - M) : 0.f;
    const float a = (lane < nsplit && ms != -INFINITY) ? __expf(ms - M) : 0.f;   // empty split: weight 0
    // denominator: the splits' weighted sums (lane = split) plus the extra tokens'
    const float den = wave_sum((lane < nsplit) ? a * ml.y : 0.f);
    if (lane == 0) {
      s_me = mx;
      s_ae = ae;
      s_den = den + ae * sm;
    }
    if (lane < kMaxSplit) s_as[lane] = a;
  }
  __syncthreads();
  // ---- weighted split outputs: thread t holds dims 4 t % dh .. + 3 -----------------------
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < CV; ++i) {
    const int e4 = t + 256 * i;
    if (e4 < ne4) {
      const float a = s_as[(4 * e4) >> ldh];
      acc.x += po[i].x * a;
      acc.y += po[i].y * a;
      acc.z += po[i].z * a;
      acc.w += po[i].w * a;
    }
  }
  *reinterpret_cast<float4*>(&red[4 * t]) = acc;   // red[e] holds dim e % dh
  __syncthreads();
  if (t < dh) {
    float num = 0.f;
#pragma unroll 8
    for (int k = t; k < 1024; k += dh) num += red[k];
    if (n_extra > 0) {
      const float me = s_me;
      float o = 0.f;
#pragma unroll
      for (int e = 0; e < kPreTok; ++e)
        if (e < n_extra) o = fmaf(__expf(lg[e] - me), pv[e], o);
#pragma unroll 4
      for (int e = kPreTok; e < n_extra; ++e) o = fmaf(__expf(lg[e] - me), load_elem(vrow(e), t), o);
      num += o * s_ae;
    }
    out[((int64_t)b * hq + h) * dh + t] = num / s_den;
  }
}

// the split merge of nsplit partials per (query head, sequence) with the extra
// full-precision tokens (sinks, optional exact window) attended beside them
template <typename T>
static void launch_combine_t(const Problem& P, const Workspace& ws, int64_t L, int nsplit, const void* q,
                             const void* sink_k, const void* sink_v, const void* win_k, const void* win_v, int s_sink,
                             int W, float* out, hipStream_t st) {
  const int need = (nsplit * P.dh + 1023) / 1024;
  auto kern = need <= 1 ? k_attn_combine<T, 1>
              : need <= 2 ? k_attn_combine<T, 2> : need <= 4 ? k_attn_combine<T, 4> : k_attn_combine<T, kCombVec>;
  hipLaunchKernelGGL(kern, dim3(P.hq, P.B), dim3(256), 0, st, (const T*)q, (const T*)sink_k, (const T*)sink_v,
                     (const T*)win_k, (const T*)win_v, ws.part_ml, ws.part_o, out, nsplit, P.hq, P.hkv, P.dh, s_sink,
                     W, L, rope_ratio(P), P.lens);
}

// ---------------------------------------------------------------------------
// explicit reconstruction: K^[b, n, :] = C^K[b, idx[b, n]] (B^K)^T (fp32 out)
// ---------------------------------------------------------------------------
// grid (ceil(m / (16 NT)), h_kv, B), four waves: wave w forms the key (w < 2)
// or value rows of NT tiles of 16 tokens over half w % 2 of head j's dims.
// Bound by latency at decode sizes (m = 1088, 8 heads: 9 MB written), so every
// basis block of a dims step is requested before the first product, and the
// basis is the A operand: a lane then holds four consecutive dims of one token
// and stores 16 bytes.  A tile's share of the basis is five times what it
// writes at rank 160, so larger m is bound by reading it from L2: one read
// serves all NT tiles.  Whole call at rank 160, 8 heads, one wave per 16 tokens
// walking both sides / NT 1 / NT 4: 11.1 / 8.9 / 8.0 us at m = 1088, 31.1 / 34.5 /
// 24.6 at 8000, 86.8 / 96.1 / 65.3 at 24000; fp32 (NT 2) 35.0 / 20.4 / 17.5 and
// 256 / 274 / 175.
template <typename T, int RBH, int NT>
__global__ __launch_bounds__(256) void k_reconstruct(
    const int32_t* __restrict__ idx_all, const T* __restrict__ bases_k, const T* __restrict__ bases_v,
    const T* __restrict__ coef_k, const T* __restrict__ coef_v, float* __restrict__ k_hat,
    float* __restrict__ v_hat, int m, int hkv, int dh, int nb, int rank, int R, int64_t L, int64_t cap,
    int bases_shared) {
  constexpr int NP = Parts<T>::n;
  const int j = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, slot = lane & 15, kg = lane >> 4;
  const int which = w >> 1, half = w & 1;
  const int Dp = hkv * dh, Dg = Dp / nb;
  const int grp = j / (hkv / nb), row0 = (j % (hkv / nb)) * dh, kb0 = grp * rank / 32;
  const int64_t boff = (bases_shared ? 0 : (int64_t)b * Dp * rank) + (int64_t)grp * Dg * rank;
  const T* cb = (which == 0 ? coef_k : coef_v) + (int64_t)b * cap * R;
  const T* bb = (which == 0 ? bases_k : bases_v) + boff;
  const int n0 = blockIdx.x * NT * 16 + slot;      // row of this lane in the first tile
  float* dst = (which == 0 ? k_hat : v_hat) + ((int64_t)b * m + n0) * Dp + (int64_t)j * dh;
  bool bad[NT];
  Op8 c[NT][RBH][NP];
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    const int n = n0 + q * 16;
    int64_t tok = (n < m) ? (int64_t)idx_all[(int64_t)b * m + n] : 0;
    bad[q] = tok < 0 || tok >= L;                  // NaN row instead of a read out of range
    if (bad[q]) tok = 0;
    const int64_t co = (tok >> 4) * 16 * (int64_t)R + (tok & 15) * 32 + kg * 8;
#pragma unroll
    for (int kb = 0; kb < RBH; ++kb) Parts<T>::load(cb + co + (int64_t)(kb0 + kb) * 512, c[q][kb]);
  }
  const int nblk = dh / 32;                        // 16-dim blocks of this wave's half
  constexpr int BST = NP == 1 ? 2 : 1;             // blocks per step (nblk is 2 or 4)
  for (int i0 = 0; i0 < nblk; i0 += BST) {
    Op8 bo[BST][RBH][NP];
#pragma unroll
    for (int u = 0; u < BST; ++u)
#pragma unroll
      for (int kb = 0; kb < RBH; ++kb)
        Parts<T>::load(bb + (int64_t)(row0 + (half * nblk + i0 + u) * 16 + slot) * rank + kb * 32 + kg * 8, bo[u][kb]);
    if constexpr (NP == 1) __builtin_amdgcn_sched_barrier(0);   // the loads stay together, ahead of the products
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int u = 0; u < BST; ++u) {
        floatx4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < RBH; ++kb) d = mfma_parts<NP, NP>(bo[u][kb], c[q][kb], d);
        if (bad[q]) d = floatx4{NAN, NAN, NAN, NAN};
        // lane holds token slot, dims 4 kg + v of the block
        if (n0 + q * 16 < m)
          *reinterpret_cast<floatx4*>(dst + (int64_t)q * 16 * Dp + (half * nblk + i0 + u) * 16 + kg * 4) = d;
      }
  }
}

// ---------------------------------------------------------------------------
// explicit attention over given fp32 rows
// ---------------------------------------------------------------------------
// grid (row splits, h_kv, B), four waves: a workgroup attends one KV head's G
// query heads to its share of the rows, in chunks of 32 with one running
// maximum per head, and leaves a split partial that k_attn_combine merges with
// the sinks.  A row's RoPE pair f sits in lane f (d_h = 128; two rows per wave
// at d_h = 64), so a wave reads whole rows, and the 8 rows x up to 4 heads of
// dot products are summed over the lanes by halving exchanges (31 instead of
// 192).  Both the key and the value rows of a chunk are requested before any
// is used.  Reading the rows bounds it (8 bytes per row element) once the
// splits fill the chip; the single workgroup per query head that it replaces,
// whose threads walked all rows of V one by one, took 334 us at m = 1088, 8 KV
// heads, against 7.3 us.
constexpr int kSaRows = 32;            // rows per chunk

// sums of N values over the 2 O lanes that differ in the bits O, O / 2, .., 1:
// while several values are left a lane keeps half of them and adds its
// partner's sums of those, then plain exchanges; the lane whose bits under 2 O
// are f ends with value f / (2 O / N) in v[0] (N <= 2 O).  Recursive, so every
// index is a constant: a loop over a shrinking count became 7000 instructions
// of selects, past what the instruction cache holds.
template <int N, int O>
__device__ __forceinline__ void lane_sums(float* v, int lane) {
  if constexpr (O > 0) {
    if constexpr (N > 1) {
      const bool up = (lane & O) != 0;
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const float keep = up ? v[i + N / 2] : v[i], send = up ? v[i] : v[i + N / 2];
        v[i] = keep + shfl_xor_f(send, O);
      }
      lane_sums<N / 2, O / 2>(v, lane);
    } else {
      v[0] += shfl_xor_f(v[0], O);
      lane_sums<1, O / 2>(v, lane);
    }
  }
}
template <typename T, int DH, int GB>
__global__ __launch_bounds__(256) void k_sparse_attn(
    const T* __restrict__ q, const int32_t* __restrict__ idx_all, const float* __restrict__ k_sel,
    const float* __restrict__ v_sel, float* __restrict__ part_ml, float* __restrict__ part_o, int m,
    int rows_per_split, int G, int hq, int hkv, int s_sink, int64_t L, double rope_ratio) {
  constexpr int HALF = DH / 2;                     // lanes per row
  constexpr int RPW = kSaRows / 4;                 // rows per wave (8)
  constexpr int PAR = 64 / HALF;                   // rows side by side in a wave
  constexpr int RPL = RPW / PAR;                   // rows per lane
  constexpr int GP = GB < 4 ? GB : 4;              // heads per reduction
  constexpr int NV = RPL * GP;                     // values per reduction (<= lanes per row)
  constexpr int NPH = 256 / DH;                    // row phases of the value pass
  const int split = blockIdx.x, j = blockIdx.y, b = blockIdx.z;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int f = lane % HALF, par = lane / HALF;
  const int Dp = hkv * DH;
  const int r_begin = split * rows_per_split, r_end = min(m, r_begin + rows_per_split);   // r_begin < m
  __shared__ float sl[GB][kSaRows];
  __shared__ float s_alpha[GB];
  __shared__ float red[NPH][GB][DH];
  const float* kb = k_sel + (int64_t)b * m * Dp + (int64_t)j * DH;
  const float* vb = v_sel + (int64_t)b * m * Dp + (int64_t)j * DH;
  const int32_t* idx = idx_all + (int64_t)b * m;
  uint64_t F[4];
  rope_freqs_fixed(rope_ratio, f, F);
  float ql[GB], qh[GB];
  {
    float c, sn;
    rope_cs_fixed(s_sink + L - 1, F[0], c, sn);
    const float inv = 1.0f / sqrtf((float)DH);
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      const int64_t qo = ((int64_t)b * hq + (int64_t)j * G + min(g, G - 1)) * DH;
      const float xl = load_elem(q, qo + f), xh = load_elem(q, qo + f + HALF);
      ql[g] = (xl * c - xh * sn) * inv;
      qh[g] = (xh * c + xl * sn) * inv;
    }
  }
  const int dim = t % DH, ph = t / DH;
  float acc[GB];
#pragma unroll
  for (int g = 0; g < GB; ++g) acc[g] = 0.f;
  // softmax state of heads w, w + 4, .. (every lane of wave w holds the same)
  constexpr int GW = (GB + 3) / 4;
  float Mr[GW], lr[GW];
#pragma unroll
  for (int i = 0; i < GW; ++i) {
    Mr[i] = -INFINITY;
    lr[i] = 0.f;
  }
  for (int r0 = r_begin; r0 < r_end; r0 += kSaRows) {
    float kl[RPL], kh[RPL], vv[kSaRows / NPH];
    int32_t pos[RPL];
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const int r = min(r0 + w * RPW + par * RPL + i, r_end - 1);
      kl[i] = kb[(int64_t)r * Dp + f];
      kh[i] = kb[(int64_t)r * Dp + f + HALF];
      pos[i] = idx[r];
    }
#pragma unroll
    for (int i = 0; i < kSaRows / NPH; ++i) vv[i] = vb[(int64_t)min(r0 + i * NPH + ph, r_end - 1) * Dp + dim];
    __builtin_amdgcn_sched_barrier(0);             // every load of the chunk is requested before any is used
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      float c, sn;
      rope_cs_fixed((int64_t)s_sink + pos[i], F[0], c, sn);
      const float a = kl[i] * c - kh[i] * sn, d = kh[i] * c + kl[i] * sn;
      kl[i] = a;
      kh[i] = d;
    }
    for (int g0 = 0; g0 < GB; g0 += GP) {
      float v[NV];
#pragma unroll
      for (int g = 0; g < GP; ++g)
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
          // g0 + g by compile-time selection (the query stays in registers)
          float a = 0.f, d = 0.f;
#pragma unroll
          for (int gg = g; gg < GB; gg += GP) {
            a = (gg == g0 + g) ? ql[gg] : a;
            d = (gg == g0 + g) ? qh[gg] : d;
          }
          v[g * RPL + i] = fmaf(a, kl[i], d * kh[i]);
        }
      lane_sums<NV, HALF / 2>(v, lane);
      constexpr int REP = HALF / NV;               // lanes that end with the same value
      const int vi = f / REP, row = w * RPW + par * RPL + vi % RPL;
      if (f % REP == 0) sl[g0 + vi / RPL][row] = (r0 + row < r_end) ? v[0] : -INFINITY;
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < GW; ++i) {
      const int g = w + 4 * i;
      if (g < GB) {
        const float x = sl[g][lane & 31];
        float mx = slot_max16(x);
        mx = fmaxf(mx, shfl_xor_f(mx, 16));
        const float mn = fmaxf(Mr[i], mx);         // finite logits: row r0 is always live; NaN rows give NaN
        const float al = (Mr[i] == -INFINITY) ? 0.f : __expf(Mr[i] - mn);
        const float p = (x == -INFINITY) ? 0.f : __expf(x - mn);
        float sm = slot_sum16(p);
        sm += shfl_xor_f(sm, 16);
        lr[i] = lr[i] * al + sm;
        Mr[i] = mn;
        if (lane < 32) sl[g][lane] = p;
        if (lane == 0) s_alpha[g] = al;
      }
    }
    lds_barrier();
    // rows past the end weigh nothing (their slots repeat the last row, whose
    // values may be infinite)
#pragma unroll
    for (int i = 0; i < kSaRows / NPH; ++i) vv[i] = (r0 + i * NPH + ph < r_end) ? vv[i] : 0.f;
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      float a = acc[g] * s_alpha[g];
#pragma unroll
      for (int i = 0; i < kSaRows / NPH; ++i) a = fmaf(sl[g][i * NPH + ph], vv[i], a);
      acc[g] = a;
    }
    lds_barrier();                                 // sl is rewritten by the next chunk
  }
#pragma unroll
  for (int g = 0; g < GB; ++g) red[ph][g][dim] = acc[g];
  __syncthreads();
  for (int i = t; i < G * DH; i += 256) {
    const int g = i / DH, d = i % DH;
    float o = 0.f;
#pragma unroll
    for (int k = 0; k < NPH; ++k) o += red[k][g][d];
    part_o[(((int64_t)b * hq + (int64_t)j * G + g) * kMaxSplit + split) * DH + d] = o;
  }
#pragma unroll
  for (int i = 0; i < GW; ++i) {
    const int g = w + 4 * i;
    if (g < G && lane == 0) {
      float* ml = part_ml + (((int64_t)b * hq + (int64_t)j * G + g) * kMaxSplit + split) * 2;
      ml[0] = Mr[i];
      ml[1] = lr[i];
    }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int choose_splits(const Problem& P, int n_proc) {
  // about two workgroups per CU over the whole batch, at least two tiles each,
  // and an index list that fits comfortably in LDS
  const int ntile = (n_proc + 15) / 16;
  const int pairs = std::max(1, P.B * P.hkv);
  int ns = std::max(1, 512 / pairs);
  ns = std::min(ns, std::max(1, ntile / 2));
  ns = std::min(ns, kMaxSplit);
  while ((ntile + ns - 1) / ns > kMaxTilesPerSplit && ns < kMaxSplit) ++ns;
  return std::max(ns, 1);
}

// per-(dtype, head dim) instantiations live in attn_split_*.hip
bool launch_split_bf16_128(const Problem&, const Workspace&, int64_t, int, int, int, const void*, const void*,
                           const void*, const void*, const void*, hipStream_t);
bool launch_split_bf16_64(const Problem&, const Workspace&, int64_t, int, int, int, const void*, const void*,
                          const void*, const void*, const void*, hipStream_t);
bool launch_split_f32_128(const Problem&, const Workspace&, int64_t, int, int, int, const void*, const void*,
                          const void*, const void*, const void*, hipStream_t);
bool launch_split_f32_64(const Problem&, const Workspace&, int64_t, int, int, int, const void*, const void*,
                         const void*, const void*, const void*, hipStream_t);

bool launch_tiles_bf16_128(const Problem&, const Workspace&, int64_t, int, int, const void*, const void*,
                           const void*, const void*, const void*, hipStream_t, int*, bool);
bool launch_tiles_bf16_64(const Problem&, const Workspace&, int64_t, int, int, const void*, const void*,
                          const void*, const void*, const void*, hipStream_t, int*, bool);

// which (G, rank) pairs the fused attention kernel is built for (asymmetric
// key / value ranks: the bf16 MFMA kernel only)
bool attention_supported(const Problem& P) {
  if (P.rank_v != P.rank)
    return P.dtype == S4R_BF16 && (P.dh == 64 || P.dh == 128) && P.G <= 8 &&
           tiles_rank_pair(P.rank / 32, P.rank_v / 32);
  const int rb = P.rank / 32;
  const bool g_ok = P.G == 1 || P.G == 2 || P.G == 4 || P.G == 7 || P.G == 8;
  // seven blocks (rank 224, the padded r = 204) only on the bf16 MFMA kernel
  const bool rb_ok = (rb >= 1 && rb <= 6) || rb == 8 || (rb == 7 && P.dtype == S4R_BF16);
  return g_ok && rb_ok && (P.dh == 64 || P.dh == 128);
}

hipError_t launch_attention(const Problem& P, const Workspace& ws, int64_t L, int m, int k_eff, const void* q,
                            const void* sink_k, const void* sink_v, const void* win_k, const void* win_v,
                            const void* bases_k, const void* bases_v, const void* coef_k, const void* coef_v,
                            float* out, hipStream_t st, hipEvent_t* t0, hipEvent_t* t1) {
  const int n_proc = win_k ? k_eff : m;      // exact window rows go to the combine kernel
  int nsplit = choose_splits(P, n_proc);
  bool ok = true;
  if (t0 && hipEventRecord(t0[0], st) != hipSuccess) return hipErrorUnknown;
  bool tiles = false;                        // bf16: the MFMA kernel when it covers the configuration
  if (n_proc > 0 && P.dtype == S4R_BF16) {
    int ns = 0;
    tiles = P.dh == 128
                ? launch_tiles_bf16_128(P, ws, L, m, n_proc, q, bases_k, bases_v, coef_k, coef_v, st, &ns, false)
                : launch_tiles_bf16_64(P, ws, L, m, n_proc, q, bases_k, bases_v, coef_k, coef_v, st, &ns, false);
    if (tiles) nsplit = ns;
  }
  if (n_proc > 0 && !tiles && P.rank_v != P.rank) return hipErrorInvalidValue;   // MFMA kernel only
  if (n_proc > 0 && !tiles) {
    if (P.dtype == S4R_BF16)
      ok = P.dh == 128 ? launch_split_bf16_128(P, ws, L, m, n_proc, nsplit, q, bases_k, bases_v, coef_k, coef_v, st)
                       : launch_split_bf16_64(P, ws, L, m, n_proc, nsplit, q, bases_k, bases_v, coef_k, coef_v, st);
    else
      ok = P.dh == 128 ? launch_split_f32_128(P, ws, L, m, n_proc, nsplit, q, bases_k, bases_v, coef_k, coef_v, st)
                       : launch_split_f32_64(P, ws, L, m, n_proc, nsplit, q, bases_k, bases_v, coef_k, coef_v, st);
  }
  if (!ok) return hipErrorInvalidValue;
  if (t1 && hipEventRecord(t1[0], st) != hipSuccess) return hipErrorUnknown;
  if (t0 && hipEventRecord(t0[1], st) != hipSuccess) return hipErrorUnknown;
  const int ns_used = n_proc > 0 ? nsplit : 0;
  if (P.dtype == S4R_BF16)
    launch_combine_t<uint16_t>(P, ws, L, ns_used, q, sink_k, sink_v, win_k, win_v, P.s, P.W, out, st);
  else
    launch_combine_t<float>(P, ws, L, ns_used, q, sink_k, sink_v, win_k, win_v, P.s, P.W, out, st);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && t1) e = hipEventRecord(t1[1], st);
  return e;
}

// full reconstruction (Appendix B.1): attention over the sinks and all L
// tokens, each reconstructed from its coefficients: the bf16 MFMA kernel in
// its every-token mode, then the split merge with the sinks
hipError_t launch_full_recon(const Problem& P, const Workspace& ws, int64_t L, const void* q, const void* sink_k,
                             const void* sink_v, const void* bases_k, const void* bases_v, const void* coef_k,
                             const void* coef_v, float* out, hipStream_t st) {
  int ns = 0;
  const bool ok =
      P.dh == 128
          ? launch_tiles_bf16_128(P, ws, L, (int)L, (int)L, q, bases_k, bases_v, coef_k, coef_v, st, &ns, true)
          : launch_tiles_bf16_64(P, ws, L, (int)L, (int)L, q, bases_k, bases_v, coef_k, coef_v, st, &ns, true);
  if (!ok) return hipErrorInvalidValue;
  launch_combine_t<uint16_t>(P, ws, L, ns, q, sink_k, sink_v, nullptr, nullptr, P.s, P.W, out, st);
  return hipGetLastError();
}

// the split merge alone (no extra full-precision tokens), for kernels that
// leave split partials in the workspace
hipError_t launch_combine_only(const Problem& P, const Workspace& ws, int64_t L, int nsplit, const void* q, float* out,
                               hipStream_t st) {
  launch_combine_t<uint16_t>(P, ws, L, nsplit, q, nullptr, nullptr, nullptr, nullptr, 0, 0, out, st);
  return hipGetLastError();
}

template <typename T, int RBH>
static void launch_rec_t(const Problem& P, int64_t L, int m, const int32_t* idx, const void* bk, const void* bv,
                         const void* ck, const void* cv, float* kh, float* vh, hipStream_t st) {
  // tiles per workgroup: as many as the registers hold (four; two of fp32 rows
  // wider than 96, three operands each), while the workgroups still cover half
  // the CUs (fp32, bound by its products: four tiles only with one per CU)
  constexpr bool one = Parts<T>::n == 1;
  int nt = one || RBH <= 3 ? 4 : 2;
  while (nt > 1 && (int64_t)((m + 16 * nt - 1) / (16 * nt)) * P.hkv * P.B < (one ? 128 : 64 * nt)) nt >>= 1;
  auto kern = nt == 1 ? k_reconstruct<T, RBH, 1> : k_reconstruct<T, RBH, 2>;
  if constexpr (one || RBH <= 3)
    if (nt == 4) kern = k_reconstruct<T, RBH, 4>;
  hipLaunchKernelGGL(kern, dim3((m + 16 * nt - 1) / (16 * nt), P.hkv, P.B), dim3(256), 0, st, idx, (const T*)bk,
                     (const T*)bv, (const T*)ck, (const T*)cv, kh, vh, m, P.hkv, P.dh, P.nb, P.rank, P.R, L, P.cap,
                     P.bases_shared);
}

template <typename T>
static bool dispatch_rec(const Problem& P, int64_t L, int m, const int32_t* idx, const void* bk, const void* bv,
                         const void* ck, const void* cv, float* kh, float* vh, hipStream_t st) {
  switch (P.rank / 32) {
    case 1: launch_rec_t<T, 1>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    case 2: launch_rec_t<T, 2>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    case 3: launch_rec_t<T, 3>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    case 4: launch_rec_t<T, 4>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    case 5: launch_rec_t<T, 5>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    case 6: launch_rec_t<T, 6>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    case 7: launch_rec_t<T, 7>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    case 8: launch_rec_t<T, 8>(P, L, m, idx, bk, bv, ck, cv, kh, vh, st); return true;
    default: return false;
  }
}

hipError_t launch_reconstruct(const Problem& P, int64_t L, int m, const int32_t* idx, const void* bases_k,
                              const void* bases_v, const void* coef_k, const void* coef_v, float* k_hat,
                              float* v_hat, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  bool ok = P.dtype == S4R_BF16
                ? dispatch_rec<uint16_t>(P, L, m, idx, bases_k, bases_v, coef_k, coef_v, k_hat, v_hat, st)
                : dispatch_rec<float>(P, L, m, idx, bases_k, bases_v, coef_k, coef_v, k_hat, v_hat, st);
  if (!ok) return hipErrorInvalidValue;
  return hipGetLastError();
}

// row splits of the explicit attention: about two workgroups per CU over the
// batch (one chunk of rows each, or fewer rows, while that leaves the chip
// idle), at most kMaxSplit
template <typename T, int DH>
static int launch_sparse_rows(const Problem& P, const Workspace& ws, int64_t L, int m, const void* q,
                              const int32_t* idx, const float* k_sel, const float* v_sel, hipStream_t st) {
  int ns = std::max(1, std::min(kMaxSplit, 512 / std::max(1, P.B * P.hkv)));
  const int rows = std::max(8, (m + ns - 1) / ns);
  ns = (m + rows - 1) / rows;
  auto kern = P.G <= 1   ? k_sparse_attn<T, DH, 1>
              : P.G <= 2 ? k_sparse_attn<T, DH, 2>
              : P.G <= 4 ? k_sparse_attn<T, DH, 4>
              : P.G <= 8 ? k_sparse_attn<T, DH, 8> : k_sparse_attn<T, DH, 16>;
  hipLaunchKernelGGL(kern, dim3(ns, P.hkv, P.B), dim3(256), 0, st, (const T*)q, idx, k_sel, v_sel, ws.part_ml,
                     ws.part_o, m, rows, P.G, P.hq, P.hkv, P.s, L, rope_ratio(P));
  return ns;
}

hipError_t launch_sparse_attn(const Problem& P, const Workspace& ws, int64_t L, int m, const void* q,
                              const void* sink_k, const void* sink_v, const int32_t* idx, const float* k_sel,
                              const float* v_sel, float* out, hipStream_t st) {
  int ns = 0;
  if (P.dtype == S4R_BF16) {
    if (m > 0)
      ns = P.dh == 128 ? launch_sparse_rows<uint16_t, 128>(P, ws, L, m, q, idx, k_sel, v_sel, st)
                       : launch_sparse_rows<uint16_t, 64>(P, ws, L, m, q, idx, k_sel, v_sel, st);
    launch_combine_t<uint16_t>(P, ws, L, ns, q, sink_k, sink_v, nullptr, nullptr, P.s, 0, out, st);
  } else {
    if (m > 0)
      ns = P.dh == 128 ? launch_sparse_rows<float, 128>(P, ws, L, m, q, idx, k_sel, v_sel, st)
                       : launch_sparse_rows<float, 64>(P, ws, L, m, q, idx, k_sel, v_sel, st);
    launch_combine_t<float>(P, ws, L, ns, q, sink_k, sink_v, nullptr, nullptr, P.s, 0, out, st);
  }
  return hipGetLastError();
}

}  // namespace s4r
