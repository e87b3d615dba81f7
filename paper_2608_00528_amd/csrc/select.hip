// Index selection of Section 3.2.3 on gfx950:
//   I_local  = [max(L - W, 0), L)
//   I_global = the k_eff = min(k, max(L - W, 0)) largest scores of
//              [0, L - W), equal scores going to the lower position
//   idx      = sorted(I_global) ++ I_local
//
// Scores are non-negative fp32, so their bit patterns (sign bit shifted out)
// order like the values;
// a candidate is the composite (key << 32) | ~position, unique, and larger
// exactly when it goes first (higher score, then lower position).
//
// A 2048-bin histogram of the top 11 key bits (built by the relevance kernel,
// k_hist_scores or the kernel itself) fixes the boundary bin b1: count(bins >
// b1) < k_eff <= count(bins >= b1).  The next 11 key bits of b1's members fix
// the boundary sub-bin b2 the same way; of the members of b2 (usually a
// handful: only exact ties share all 22 bits) the need3 largest composites are
// ranked exactly.
//   k_select_one       short caches: one workgroup of 1024 threads per sequence
//                      does all of it with the keys in registers;
//   k_select_classify, longer ones, one workgroup per 2048 positions each: the
//   k_select_finish    first marks the positions above b1 in a bitmap, counts
//                      them per chunk, lists the chunk's b1 candidates and
//                      adds their next 11 key bits to a second histogram
//                      (global atomics); in the second every workgroup derives
//                      the rule, counts what is chosen in the chunks before its
//                      own and writes its own chunk's positions in ascending
//                      order.
// All of them are bound by latency (a launch, a first read, and a chain of
// block-wide steps), so scans and sums use DPP, per-wave counts come from
// ballots, and barriers are few: classify and finish 6.7 + 8.6 -> 5.2 + 5.4 us
// at 4 x 128k (k = 2048), 7.0 + 13.5 -> 5.5 + 6.3 us at 120k (k = 24k), where
// every candidate had been looked up by a binary search and counted by atomics
// on its chunk's counter.
// Integer work on the given scores: bit-exact and deterministic.
#include "s4r_device.h"
#include "s4r_internal.h"
#include "select_key.h"

namespace s4r {

constexpr int kSelThreads = 256;
constexpr int kSelPer = kSelChunk / kSelThreads;   // consecutive positions per thread (8)
constexpr int kS3Cap = 1024;                       // level-3 candidates ranked by counting
constexpr int kSubShift = kHistShift - 11;         // the next 11 key bits (level 2)
constexpr uint32_t kLow10 = (1u << kSubShift) - 1; // the key bits below them

// inclusive prefix sum over the wave's lanes: row shifts within 16 lanes, then
// the last lane of each row broadcast to the rows after it
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);   // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);   // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);   // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);   // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // row_bcast:31
  return x;
}
__device__ __forceinline__ uint32_t wave_total(uint32_t scanned) {
  return (uint32_t)__builtin_amdgcn_readlane((int)scanned, 63);
}

// block-wide exclusive prefix sum over NT threads (one barrier; each call needs
// its own scratch of NT / 64 words, which the next call must not reuse before
// another barrier); returns the block total
template <int NT>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* scratch, uint32_t& excl) {
  constexpr int NW = NT / 64;
  static_assert(NW <= 16, "the wave totals fit one DPP row");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t x = wave_scan(v);
  if (lane == 63) scratch[wave] = x;
  lds_barrier();
  uint32_t t = (lane & 15) < NW ? scratch[lane & 15] : 0u;   // every row of the wave: the wave totals
  t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x111, 0xF, 0xF, false);
  t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x112, 0xF, 0xF, false);
  t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x114, 0xF, 0xF, false);
  t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x118, 0xF, 0xF, false);
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)t, NW - 1);
  const int w = __builtin_amdgcn_readfirstlane(wave);
  const uint32_t before = w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)t, w - 1) : 0u;
  excl = before + x - v;
  return total;
}

// boundary bin of a histogram whose bins are held descending, PER per thread
// (thread t: bins nbins - 1 - (t PER + i)): the highest bin b with
// count(bins >= b) >= kk; `above` = count(bins > b).  Two barriers; `s` is
// NT / 64 + 2 words of LDS used by this call only.
template <int NT, int PER>
__device__ __forceinline__ void find_boundary(const uint32_t (&cnt)[PER], int nbins, uint32_t kk, uint32_t* s, int& bin,
                                              uint32_t& above) {
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) sum += cnt[i];
  uint32_t excl;
  block_scan<NT>(sum, s, excl);                    // count strictly above this thread's bins
  uint32_t* res = s + NT / 64;
  if (excl < kk && excl + sum >= kk) {
    uint32_t run = excl;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (run < kk && run + cnt[i] >= kk) {
        res[0] = (uint32_t)(nbins - 1 - ((int)threadIdx.x * PER + i));
        res[1] = run;
      }
      run += cnt[i];
    }
  }
  lds_barrier();
  bin = (int)res[0];
  above = res[1];
}

// the thread's PER bins (descending) of a 2048-bin histogram held as NC copies
// in memory, summed
template <int PER, int NC>
__device__ __forceinline__ void load_bins(const uint32_t* __restrict__ hist, int nc, uint32_t (&cnt)[PER]) {
  const int lo = kHistBins - PER * ((int)threadIdx.x + 1);
  uint32_t v[NC][PER];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const uint32_t* hp = hist + min(c, nc - 1) * kHistBins + lo;
    if constexpr (PER % 4 == 0) {
#pragma unroll
      for (int i = 0; i < PER; i += 4) *reinterpret_cast<uint4*>(&v[c][i]) = *reinterpret_cast<const uint4*>(hp + i);
    } else {
#pragma unroll
      for (int i = 0; i < PER; i += 2) *reinterpret_cast<uint2*>(&v[c][i]) = *reinterpret_cast<const uint2*>(hp + i);
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    cnt[i] = 0u;
#pragma unroll
    for (int c = 0; c < NC; ++c) cnt[i] += c < nc ? v[c][PER - 1 - i] : 0u;
  }
}

// ---------------------------------------------------------------------------
// one workgroup per sequence
// ---------------------------------------------------------------------------
// EPT keys per thread: wave w holds positions 64 (16 i + w) + lane, i < EPT, so
// a ballot is two words of the bitmap (lane i of the wave keeps iteration i's).
// OWN: the top-level histogram is counted here (the standalone selection)
// instead of read from the relevance kernel's copies.
constexpr int kOneThreads = 1024;
// positions up to which it is used.  In the step it replaces two kernels of
// about 10 us together: 5.4 us at 4k and 8.5 at 16k, but 13.1 at 32k, where one
// CU's passes over the keys cost more than a second launch.  The standalone
// selection would take four kernels (17 us and four launches): 16.6 us at 32k.
constexpr int kOneMax = 16 * kOneThreads, kOneOwnMax = 32 * kOneThreads;

template <int EPT, bool OWN>
__global__ __launch_bounds__(kOneThreads) void k_select_one(const float* __restrict__ scores, int64_t score_stride,
                                                            const uint32_t* __restrict__ hist_all, int hist_nc,
                                                            int32_t* __restrict__ idx_all, int32_t* __restrict__ idx_copy,
                                                            int64_t idx_stride, int L, int W, int k, Lens lens,
                                                            int key_shift) {
  constexpr int NW = kOneThreads / 64;
  constexpr int NBLK = EPT * NW;                   // 64-position blocks
  const int b = blockIdx.x;
  L = (int)len_of(lens, b, L);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n_hist = max(L - W, 0);
  const int k_eff = min(k, n_hist);
  int32_t* idx = idx_all + (int64_t)b * idx_stride;
  int32_t* idx2 = idx_copy ? idx_copy + (int64_t)b * idx_stride : nullptr;
  for (int i = t; i < L - n_hist; i += kOneThreads) {
    idx[k_eff + i] = n_hist + i;
    if (idx2) idx2[k_eff + i] = n_hist + i;
  }
  if (k_eff == 0) return;

  __shared__ uint32_t h[kHistBins];
  __shared__ uint32_t bitmap[2 * NBLK];
  __shared__ uint64_t s3[kS3Cap];
  __shared__ uint32_t sb1[NW + 2], sb2[NW + 2], sb3[NW + 2], sc1[NW], sc2[NW];
  __shared__ uint32_t s_n3, s_slot;

  const float* sc = scores + (int64_t)b * score_stride;
  float v[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) v[i] = sc[min((i * NW + w) * 64 + lane, n_hist - 1)];
  uint32_t cnt[2];
  if constexpr (!OWN) load_bins<2, kHistCopies>(hist_all + (int64_t)b * kHistStride, hist_nc, cnt);
  reinterpret_cast<uint2*>(h)[t] = make_uint2(0u, 0u);
  if (t == 0) {
    s_n3 = 0u;
    s_slot = 0u;
  }
  // keys are even (a bit or two were shifted out at the bottom): 1 marks a
  // position past the end, which no comparison below takes for a member
  uint32_t key[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i)
    key[i] = (i * NW + w) * 64 + lane < n_hist ? selection_key_shift(v[i], key_shift) : 1u;
  auto live = [](uint32_t x) { return (x & 1u) == 0u; };
  if constexpr (OWN) {
    lds_barrier();
#pragma unroll
    for (int i = 0; i < EPT; ++i)
      if (live(key[i])) atomicAdd(&h[key[i] >> kHistShift], 1u);
    lds_barrier();
    const uint2 c2 = reinterpret_cast<const uint2*>(h)[kOneThreads - 1 - t];
    cnt[0] = c2.y;
    cnt[1] = c2.x;
    lds_barrier();
    reinterpret_cast<uint2*>(h)[t] = make_uint2(0u, 0u);
  }
  int b1, b2;
  uint32_t above1, above2;
  find_boundary<kOneThreads>(cnt, kHistBins, (uint32_t)k_eff, sb1, b1, above1);   // (its barriers also cover h)

  // ---- members of b1: their next 11 bits counted ------------------------------------------
#pragma unroll
  for (int i = 0; i < EPT; ++i)
    if (live(key[i]) && (int)(key[i] >> kHistShift) == b1)
      atomicAdd(&h[(key[i] >> kSubShift) & (kHistBins - 1)], 1u);
  lds_barrier();
  {
    const uint2 c2 = reinterpret_cast<const uint2*>(h)[kOneThreads - 1 - t];
    cnt[0] = c2.y;
    cnt[1] = c2.x;
  }
  const uint32_t need = (uint32_t)k_eff - above1;  // >= 1
  find_boundary<kOneThreads>(cnt, kHistBins, need, sb2, b2, above2);
  const uint32_t need3 = need - above2;            // >= 1, taken from sub-bin b2

  // ---- above sub-bin b2: chosen; members of b2 (bit i of mem: key i) to level 3 ------------
  const uint32_t top = ((uint32_t)b1 << 11) | (uint32_t)b2;   // the 22 bits of sub-bin b2
  uint32_t mlo = 0u, mhi = 0u, mem = 0u;           // lane i of mlo, mhi: the chosen of block (i, w)
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const uint32_t k22 = key[i] >> kSubShift;
    const uint64_t m = __ballot(k22 > top);        // (a position past the end has k22 = 0)
    mlo = (lane == i) ? (uint32_t)m : mlo;
    mhi = (lane == i) ? (uint32_t)(m >> 32) : mhi;
    mem |= (k22 == top && live(key[i])) ? 1u << i : 0u;
  }
  if (lane < EPT) reinterpret_cast<uint2*>(bitmap)[lane * NW + w] = make_uint2(mlo, mhi);
  if (mem) atomicAdd(&s_n3, (uint32_t)__popc(mem));
  lds_barrier();
  const uint32_t n3 = s_n3;
  if (n3 <= (uint32_t)kS3Cap) {
    // listed with their scores read again (few lanes have any)
    uint32_t rest = mem;
    while (__ballot(rest != 0u)) {
      const bool has = rest != 0u;
      const int i = has ? __ffs(rest) - 1 : 0;
      const int x = (i * NW + w) * 64 + lane;
      const uint32_t slot = wave_append(&s_slot, has);
      if (has)
        s3[slot] = ((uint64_t)(selection_key_shift(sc[x], key_shift) & kLow10) << 32) | (0xFFFFFFFFu - (uint32_t)x);
      rest &= rest - 1;
    }
  }
  lds_barrier();
  if (n3 <= (uint32_t)kS3Cap) {
    // exact rank among the level-3 members by counting larger composites
    if (t < (int)n3) {
      const uint64_t x = s3[t];
      uint32_t rank = 0;
      for (uint32_t j = 0; j < n3; ++j) rank += (s3[j] > x) ? 1u : 0u;
      if (rank < need3) {
        const uint32_t pos = 0xFFFFFFFFu - (uint32_t)x;
        atomicOr(&bitmap[pos >> 5], 1u << (pos & 31));
      }
    }
  } else {
    // many members: the boundary of their last 10 bits, then the lowest
    // positions of those that share all 32
    reinterpret_cast<uint2*>(h)[t] = make_uint2(0u, 0u);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < EPT; ++i)
      if (live(key[i]) && (key[i] >> kSubShift) == top) atomicAdd(&h[key[i] & kLow10], 1u);
    lds_barrier();
    uint32_t c1[1] = {h[kLow10 - t]};
    int b3;
    uint32_t above3;
    find_boundary<kOneThreads>(c1, (int)kLow10 + 1, need3, sb3, b3, above3);
    const uint32_t need4 = need3 - above3, last = (top << kSubShift) | (uint32_t)b3;
    uint32_t glo = 0u, ghi = 0u, elo = 0u, ehi = 0u;
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const uint64_t g = __ballot(live(key[i]) && (key[i] >> kSubShift) == top && key[i] > last);
      const uint64_t e = __ballot(key[i] == last);
      glo = (lane == i) ? (uint32_t)g : glo;
      ghi = (lane == i) ? (uint32_t)(g >> 32) : ghi;
      elo = (lane == i) ? (uint32_t)e : elo;
      ehi = (lane == i) ? (uint32_t)(e >> 32) : ehi;
    }
    if (lane < EPT) h[lane * NW + w] = (uint32_t)(__popc(elo) + __popc(ehi));   // ties per block, in position order
    lds_barrier();
    uint32_t pre;
    block_scan<kOneThreads>(t < NBLK ? h[t] : 0u, sc1, pre);
    if (t < NBLK) h[t] = pre;
    lds_barrier();
    if (lane < EPT) {
      uint32_t keep = need4 > h[lane * NW + w] ? need4 - h[lane * NW + w] : 0u;
      uint64_t e = ((uint64_t)ehi << 32) | elo, out = 0;
      while (e && keep) {
        out |= e & (~e + 1);
        e &= e - 1;
        --keep;
      }
      out |= ((uint64_t)ghi << 32) | glo;
      bitmap[2 * (lane * NW + w)] |= (uint32_t)out;
      bitmap[2 * (lane * NW + w) + 1] |= (uint32_t)(out >> 32);
    }
  }
  lds_barrier();
  // ---- positions ascending: word t of the bitmap ------------------------------------------
  uint32_t word = t < 2 * NBLK ? bitmap[min(t, 2 * NBLK - 1)] : 0u, pos;
  block_scan<kOneThreads>((uint32_t)__popc(word), sc2, pos);
  while (word) {
    const int bit = __ffs(word) - 1;
    word &= word - 1;
    idx[pos] = t * 32 + bit;
    if (idx2) idx2[pos] = t * 32 + bit;
    ++pos;
  }
}

// ---------------------------------------------------------------------------
// classify: one workgroup per 2048 positions
// ---------------------------------------------------------------------------
// A candidate is one word: the 21 key bits below the top 11, then the position
// within its chunk (descending), so larger goes first within the chunk.
constexpr int kPosBits = 11;
static_assert(kSelChunk == 1 << kPosBits, "candidate words");

template <int NC>   // copies of the top-level histogram (a power of two, at most kHistCopies)
__global__ __launch_bounds__(kSelThreads) void k_select_classify(
    const float* __restrict__ scores, int64_t score_stride, uint32_t* __restrict__ hist_all,
    uint32_t* __restrict__ cand_all, uint32_t* __restrict__ bitmap_all, uint32_t* __restrict__ cand_count,
    uint32_t* __restrict__ above_count, uint32_t* __restrict__ sel_info, int64_t cand_stride, int64_t cnt_stride,
    int64_t cap, int L, int W, int k, Lens lens, int key_shift) {
  const int b = blockIdx.y, c = blockIdx.x;
  L = (int)len_of(lens, b, L);
  const int t = threadIdx.x, lane = t & 63;
  const int n_hist = max(L - W, 0);
  const int k_eff = min(k, n_hist);
  if (k_eff == 0 || c * kSelChunk >= n_hist) return;   // (a shorter sequence of a ragged batch)
  uint32_t* hist1 = hist_all + (int64_t)b * kHistStride;
  uint32_t* hist2 = hist1 + kHistCopies * kHistBins;
  uint32_t* cand = cand_all + (int64_t)b * cand_stride + (int64_t)c * kSelChunk;
  const float* sc = scores + (int64_t)b * score_stride;
  const int c0 = c * kSelChunk;

  __shared__ uint32_t sb[kSelThreads / 64 + 2], ss[kSelThreads / 64];
  __shared__ uint32_t h2[kHistBins];
  // this thread's 8 consecutive scores (unguarded: masked below)
  float v[kSelPer];
#pragma unroll
  for (int i = 0; i < kSelPer; ++i) v[i] = sc[min(c0 + t * kSelPer + i, n_hist - 1)];
  uint32_t cnt[kHistBins / kSelThreads];
  load_bins<kHistBins / kSelThreads, NC>(hist1, NC, cnt);
  for (int i = t; i < kHistBins / 4; i += kSelThreads) reinterpret_cast<uint4*>(h2)[i] = make_uint4(0u, 0u, 0u, 0u);
  int b1;
  uint32_t above1;
  find_boundary<kSelThreads>(cnt, kHistBins, (uint32_t)k_eff, sb, b1, above1);
  if (c == 0 && t == 0) {
    sel_info[b * 4 + 0] = (uint32_t)b1;
    sel_info[b * 4 + 1] = above1;
  }
  uint32_t mask8 = 0u, cmask = 0u;
  uint32_t key[kSelPer];
#pragma unroll
  for (int i = 0; i < kSelPer; ++i) {
    key[i] = selection_key_shift(v[i], key_shift);
    const int bin = (int)(key[i] >> kHistShift);
    const bool valid = c0 + t * kSelPer + i < n_hist;
    mask8 |= (valid && bin > b1) ? 1u << i : 0u;
    cmask |= (valid && bin == b1) ? 1u << i : 0u;
  }
  // both counts in one scan (a chunk has 2048 positions)
  uint32_t excl;
  const uint32_t total = block_scan<kSelThreads>((uint32_t)__popc(mask8) | ((uint32_t)__popc(cmask) << 16), ss, excl);
  uint32_t slot = excl >> 16;
#pragma unroll
  for (int i = 0; i < kSelPer; ++i) {
    if ((cmask >> i) & 1u) {
      cand[slot++] = (key[i] << kPosBits) | (uint32_t)(kSelChunk - 1 - (t * kSelPer + i));
      atomicAdd(&h2[(key[i] >> kSubShift) & (kHistBins - 1)], 1u);
    }
  }
  // a bitmap word covers 4 threads' bytes: lane 4q gathers lanes 4q..4q+3
  const uint32_t m1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mask8, 0xF9, 0xF, 0xF, false),   // quad_perm [1,2,3,3]
                 m2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mask8, 0xFE, 0xF, 0xF, false),   // [2,3,3,3]
                 m3 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mask8, 0xFF, 0xF, 0xF, false);   // [3,3,3,3]
  const uint32_t word = mask8 | (m1 << 8) | (m2 << 16) | (m3 << 24);
  const int wi = t >> 2;                                // word index within the chunk
  if ((lane & 3) == 0 && c0 + wi * 32 < n_hist) bitmap_all[b * bitmap_words(cap) + c0 / 32 + wi] = word;
  if (t == 0) {
    above_count[(int64_t)b * cnt_stride + c] = total & 0xFFFFu;
    cand_count[(int64_t)b * cnt_stride + c] = total >> 16;
  }
  lds_barrier();                                        // h2 complete
  for (int i = t; i < kHistBins; i += kSelThreads) {
    const uint32_t n = h2[i];
    if (n) atomicAdd(&hist2[i], n);
  }
}

// ---------------------------------------------------------------------------
// finish: one workgroup per 2048 positions
// ---------------------------------------------------------------------------
// Wave w goes over the candidate lists of chunks w, w + 8, ..: a ballot counts
// what a chunk has above b2, so the chunks before this one need no counters.
constexpr int kFinThreads = 512;
constexpr int kFinWaves = kFinThreads / 64;
constexpr int kFinBatch = 4;                            // chunks whose lists are requested together

__global__ __launch_bounds__(kFinThreads) void k_select_finish(
    const uint32_t* __restrict__ hist_all, const uint32_t* __restrict__ cand_all,
    const uint32_t* __restrict__ bitmap_all, const uint32_t* __restrict__ cand_count,
    const uint32_t* __restrict__ above_count, const uint32_t* __restrict__ sel_info, int32_t* __restrict__ idx_all,
    int32_t* __restrict__ idx_copy, int64_t idx_stride, int64_t cand_stride, int64_t cnt_stride, int64_t cap, int L,
    int W, int k, Lens lens) {
  const int b = blockIdx.y, c = blockIdx.x;
  L = (int)len_of(lens, b, L);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n_hist = max(L - W, 0);
  const int k_eff = min(k, n_hist);
  const int nch = (n_hist + kSelChunk - 1) / kSelChunk;
  int32_t* idx = idx_all + (int64_t)b * idx_stride;
  int32_t* idx2 = idx_copy ? idx_copy + (int64_t)b * idx_stride : nullptr;
  // the window goes to the workgroup of the last chunk (chunk 0 when there is none)
  if (c == max(nch, 1) - 1) {
    for (int i = t; i < L - n_hist; i += kFinThreads) {
      idx[k_eff + i] = n_hist + i;
      if (idx2) idx2[k_eff + i] = n_hist + i;
    }
  }
  if (k_eff == 0 || c >= max(nch, 1)) return;          // (a shorter sequence of a ragged batch)
  const uint32_t* cand_b = cand_all + (int64_t)b * cand_stride;
  const uint32_t* ccnt = cand_count + (int64_t)b * cnt_stride;
  const uint32_t* acnt = above_count + (int64_t)b * cnt_stride;

  __shared__ uint32_t sb[kFinWaves + 2], sb3[kFinWaves + 2];
  __shared__ uint64_t s3[kS3Cap];
  __shared__ uint32_t own[kSelChunk / 32];
  __shared__ uint32_t s_n3, s_before;
  __shared__ uint32_t h3[kLow10 + 1];

  // ---- every load the workgroup needs first, issued together ---------------------------
  const uint32_t above1 = sel_info[b * 4 + 1];
  uint32_t ncand = ccnt[min(w + kFinWaves * lane, nch - 1)];   // chunks w, w + 8, .. of this wave
  uint32_t nab = t < c ? acnt[t] : 0u;
  uint32_t cnt[kHistBins / kFinThreads];
  load_bins<kHistBins / kFinThreads, 1>(hist_all + (int64_t)b * kHistStride + kHistCopies * kHistBins, 1, cnt);
  const int wbase = c * (kSelChunk / 32);
  const int nwords = (n_hist + 31) / 32;
  if (t < kSelChunk / 32) {
    const uint32_t x = bitmap_all[b * bitmap_words(cap) + min(wbase + t, nwords - 1)];
    own[t] = (wbase + t < nwords) ? x : 0u;
  }
  if (t == 0) {
    s_n3 = 0u;
    s_before = 0u;
  }
  for (int g = t + kFinThreads; g < c; g += kFinThreads) nab += acnt[g];
  const uint32_t need = (uint32_t)k_eff - above1;        // >= 1
  int b2;
  uint32_t above2;
  find_boundary<kFinThreads>(cnt, kHistBins, need, sb, b2, above2);   // (its barriers cover own and the counters)
  const uint32_t need3 = need - above2;                  // >= 1, taken from sub-bin b2

  // f(word, chunk, live) over every candidate, whole waves
  auto for_candidates = [&](auto f) __attribute__((always_inline)) {
    for (int j0 = 0; w + kFinWaves * j0 < nch; j0 += 64) {
      const uint32_t nc = j0 == 0 ? ncand : ccnt[min(w + kFinWaves * (j0 + lane), nch - 1)];
      for (int j = 0; j < 64 && w + kFinWaves * (j0 + j) < nch; j += kFinBatch) {
        uint32_t r[kFinBatch];
        int n[kFinBatch];
#pragma unroll
        for (int q = 0; q < kFinBatch; ++q) {
          const int g = w + kFinWaves * (j0 + j + q);
          n[q] = g < nch ? (int)__builtin_amdgcn_readlane((int)nc, j + q) : 0;
          r[q] = cand_b[(int64_t)min(g, nch - 1) * kSelChunk + min(lane, max(n[q] - 1, 0))];
        }
#pragma unroll
        for (int q = 0; q < kFinBatch; ++q) {
          const int g = w + kFinWaves * (j0 + j + q);
          f(r[q], g, lane < n[q]);
          for (int i = 64; i < n[q]; i += 64) {
            const uint32_t x = cand_b[(int64_t)g * kSelChunk + min(i + lane, n[q] - 1)];
            f(x, g, i + lane < n[q]);
          }
        }
      }
    }
  };
  // a chosen candidate: counted if its chunk comes before this one, marked in this one
  auto mark = [&](int x) {
    if (x < c * kSelChunk)
      atomicAdd(&s_before, 1u);
    else if (x < (c + 1) * kSelChunk)
      atomicOr(&own[(x % kSelChunk) >> 5], 1u << (x & 31));
  };
  // position of a candidate word of chunk g
  auto pos_of = [](uint32_t x, int g) { return g * kSelChunk + (kSelChunk - 1 - (int)(x & (kSelChunk - 1))); };
  uint32_t before = 0;                                   // uniform per wave
  for_candidates([&](uint32_t x, int g, bool live) __attribute__((always_inline)) {
    const int sub = (int)(x >> (kPosBits + kSubShift));
    const uint64_t m = __ballot(live && sub > b2);
    if (g < c)
      before += (uint32_t)__popcll(m);
    else if (g == c && live && sub > b2)
      mark(pos_of(x, g));
    const bool lev3 = live && sub == b2;
    const uint32_t slot = wave_append(&s_n3, lev3);
    if (lev3 && slot < (uint32_t)kS3Cap)
      s3[slot] = ((uint64_t)((x >> kPosBits) & kLow10) << 32) | (0xFFFFFFFFu - (uint32_t)pos_of(x, g));
  });
  {
    const uint32_t sum = before + wave_total(wave_scan(nab));
    if (lane == 0 && sum) atomicAdd(&s_before, sum);
  }
  lds_barrier();
  const uint32_t n3 = s_n3;
  if (n3 <= (uint32_t)kS3Cap) {
    // exact rank among the level-3 candidates by counting larger composites
    for (int i = t; i < (int)n3; i += kFinThreads) {
      const uint64_t x = s3[i];
      uint32_t rank = 0;
      for (uint32_t j = 0; j < n3; ++j) rank += (s3[j] > x) ? 1u : 0u;
      if (rank < need3) mark((int)(0xFFFFFFFFu - (uint32_t)x));
    }
  } else {
    // many members: the boundary of their last 10 bits, then the lowest
    // positions of those that share all 32 bits: a chunk's share of them is
    // what the chunks before it leave
    for (int i = t; i <= (int)kLow10; i += kFinThreads) h3[i] = 0u;
    lds_barrier();
    for_candidates([&](uint32_t x, int, bool live) __attribute__((always_inline)) {
      if (live && (int)(x >> (kPosBits + kSubShift)) == b2) atomicAdd(&h3[(x >> kPosBits) & kLow10], 1u);
    });
    lds_barrier();
    uint32_t c2[2] = {h3[kLow10 - 2 * t], h3[kLow10 - 2 * t - 1]};
    int b3;
    uint32_t above3;
    find_boundary<kFinThreads>(c2, (int)kLow10 + 1, need3, sb3, b3, above3);
    const uint32_t need4 = need3 - above3;
    const uint32_t last = ((uint32_t)b2 << kSubShift) | (uint32_t)b3;   // the 21 bits
    // ties before this chunk (s_n3) and within it (word bitmap h3)
    if (t == 0) s_n3 = 0u;
    if (t < kSelChunk / 32) h3[t] = 0u;
    lds_barrier();
    for_candidates([&](uint32_t x, int g, bool live) __attribute__((always_inline)) {
      const uint32_t k21 = x >> kPosBits;
      if (live && k21 > last && (k21 >> kSubShift) == (uint32_t)b2) mark(pos_of(x, g));
      const uint64_t e = __ballot(live && k21 == last);
      if (g < c) {
        if (lane == 0 && e) atomicAdd(&s_n3, (uint32_t)__popcll(e));
      } else if (g == c && live && k21 == last) {
        const int p = pos_of(x, g) % kSelChunk;
        atomicOr(&h3[p >> 5], 1u << (p & 31));
      }
    });
    lds_barrier();
    const uint32_t ties = s_n3;
    if (t == 0) atomicAdd(&s_before, min(ties, need4));
    if (w == 0) {
      uint32_t tw = h3[lane];
      const uint32_t pre = wave_scan((uint32_t)__popc(tw)) - (uint32_t)__popc(tw) + ties;
      uint32_t keep = need4 > pre ? need4 - pre : 0u, out = 0u;
      while (tw && keep) {
        out |= tw & (~tw + 1);
        tw &= tw - 1;
        --keep;
      }
      own[lane] |= out;
    }
  }
  lds_barrier();

  // ---- this chunk's positions, ascending: thread t has positions 4 t .. 4 t + 3 -----------
  const uint32_t wv = own[lane];                          // every wave scans the 64 words
  const uint32_t pre = wave_scan((uint32_t)__popc(wv)) - (uint32_t)__popc(wv);
  const int wi = t >> 3, sh = (t & 7) * 4;
  const uint32_t word = (uint32_t)__shfl((int)wv, wi);
  uint32_t pos = s_before + (uint32_t)__shfl((int)pre, wi) + (uint32_t)__popc(word & ((1u << sh) - 1u));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if ((word >> (sh + i)) & 1u) {
      const int32_t p = (int32_t)(c * kSelChunk + 4 * t + i);
      idx[pos] = p;
      if (idx2) idx2[pos] = p;
      ++pos;
    }
  }
}

template <bool OWN>
static void launch_one(const Problem& P, const Workspace& ws, int64_t L, int64_t n_hist, int m, const float* scores,
                       int64_t score_stride, int32_t* idx, int32_t* idx_copy, int key_shift, int hist_nc,
                       hipStream_t st) {
  auto kern = n_hist <= 4 * kOneThreads ? k_select_one<4, OWN>
              : n_hist <= 8 * kOneThreads ? k_select_one<8, OWN> : k_select_one<16, OWN>;
  if constexpr (OWN)
    if (n_hist > kOneMax) kern = k_select_one<32, OWN>;
  hipLaunchKernelGGL(kern, dim3(P.B), dim3(kOneThreads), 0, st, scores, score_stride, ws.hist, hist_nc, idx, idx_copy,
                     (int64_t)m, (int)L, P.W, P.k, P.lens, key_shift);
}

// selection over caller-given scores: their histogram first where the
// selection does not count it itself
hipError_t launch_select(const Problem& P, const Workspace& ws, int64_t L, const float* scores,
                         int64_t score_stride, int32_t* idx, int32_t* idx_copy, hipStream_t st) {
  const int64_t n_hist = std::max<int64_t>(L - P.W, 0);
  if (n_hist <= kOneOwnMax) {
    const int m = (int)(std::min<int64_t>(P.k, n_hist) + std::min<int64_t>(P.W, L));
    launch_one<true>(P, ws, L, n_hist, m, scores, score_stride, idx, idx_copy, 1, 1, st);
    return hipGetLastError();
  }
  const hipError_t e = launch_hist_only(P, ws, L, scores, st);
  if (e != hipSuccess) return e;
  const int ng = (int)((n_hist + kHistChunk - 1) / kHistChunk);   // k_hist_scores' workgroups
  return launch_select_keyed(P, ws, L, scores, score_stride, idx, idx_copy, 1, hist_copies(ng), st);
}

hipError_t launch_select_keyed(const Problem& P, const Workspace& ws, int64_t L, const float* scores,
                               int64_t score_stride, int32_t* idx, int32_t* idx_copy, int key_shift, int hist_nc,
                               hipStream_t st) {
  const int64_t n_hist = std::max<int64_t>(L - P.W, 0);
  const int m = (int)(std::min<int64_t>(P.k, n_hist) + std::min<int64_t>(P.W, L));
  const int nch = (int)((n_hist + kSelChunk - 1) / kSelChunk);
  if (n_hist <= kOneMax) {
    launch_one<false>(P, ws, L, n_hist, m, scores, score_stride, idx, idx_copy, key_shift, hist_nc, st);
    return hipGetLastError();
  }
  if (std::min<int64_t>(P.k, n_hist) > 0) {
    static_assert(kHistCopies == 8, "classify instances for 1, 2, 4 and 8 copies");
    auto cls = hist_nc == 1 ? k_select_classify<1>
               : hist_nc == 2 ? k_select_classify<2> : hist_nc == 4 ? k_select_classify<4> : k_select_classify<8>;
    hipLaunchKernelGGL(cls, dim3(nch, P.B), dim3(kSelThreads), 0, st, scores, score_stride, ws.hist, ws.cand,
                       ws.bitmap, ws.cand_count, ws.above_count, ws.sel_info, cand_stride(P), sel_groups_max(P), P.cap,
                       (int)L, P.W, P.k, P.lens, key_shift);
  }
  hipLaunchKernelGGL(k_select_finish, dim3(nch, P.B), dim3(kFinThreads), 0, st, ws.hist, ws.cand, ws.bitmap,
                     ws.cand_count, ws.above_count, ws.sel_info, idx, idx_copy, (int64_t)m, cand_stride(P),
                     sel_groups_max(P), P.cap, (int)L, P.W, P.k, P.lens);
  return hipGetLastError();
}

}  // namespace s4r
