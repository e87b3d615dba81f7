// Bulk projection of the prefill stage (Section 3.1, the coefficient
// equation): C = S B for every non-sink prompt row, per basis group, written
// into the tiled coefficient cache (bf16 storage).
//
// k_transpose_bases first writes every basis group transposed, [column][dim],
// into the workspace.  k_prefill_project: grid (128-row blocks, basis group x
// {key, value}, sequence), 4 waves; wave w owns 2 tiles of 16 rows and walks
// the group's dims 64 at a time.  The product runs on bf16 MFMA 16x16x32 with
// fp32 accumulation in the MFMA accumulators: A = the transposed basis slice
// (one 16-byte LDS read per operand), brought into a ring of three LDS buffers
// by 16-byte global->LDS loads two steps ahead, B = the prompt rows as loaded
// (lane: row l % 16, dims 8 (l / 16) .. + 7 of a 32-dim block), two steps ahead
// in registers, so a lane ends with four consecutive columns of one row and
// stores 8 bytes.  bf16 inputs make every product exact; the fp32 sums are
// rounded once to bf16.
//
// Bound by reading the rows (2 bytes per raw element; 4 x 131072 rows of K and
// V at Dp = 1024: 2.15 GB).  A whole 128-byte line of every row is requested
// per step and 64 KB per CU are in flight; with 64 bytes of a row one step
// ahead, 2-byte stores and two-way conflicts on the slice reads the same grid
// ran at 3.5 TB/s: 704 -> 547 us (4.5 TB/s) at that shape, rank 160.
#include <type_traits>

#include "s4r_device.h"
#include "s4r_internal.h"

namespace s4r {

constexpr int kPfWaves = 4;
constexpr int kPfTiles = 2;                       // 16-row tiles per wave
constexpr int kPfRows = kPfWaves * kPfTiles * 16;  // rows per workgroup
constexpr int kPfStep = 64;                       // dims per step (Dp / basis_groups is a multiple of 64)

// s_waitcnt vmcnt(N) alone (gfx9 encoding: expcnt and lgkmcnt not waited)
template <int N>
__device__ __forceinline__ void pf_wait_vmcnt() {
  static_assert(N >= 0 && N < 16, "small counts only");
  __builtin_amdgcn_s_waitcnt(N | (7 << 4) | (15 << 8));
}

// bases [B|1][nb][Dg][rank] -> bt [B][2][nb][rank][Dg]: grid (Dg / 32, 2 nb, B),
// one 32-row x rank block per workgroup through LDS, 16 bytes per access on
// both sides (element accesses with a division each took 13.6 us)
__global__ __launch_bounds__(256) void k_transpose_bases(const uint16_t* __restrict__ bases_k,
                                                         const uint16_t* __restrict__ bases_v,
                                                         uint16_t* __restrict__ bt, int Dg, int nb, int rank,
                                                         int bases_shared) {
  const int d0 = blockIdx.x * 32, gz = blockIdx.y, b = blockIdx.z;
  const int grp = gz >> 1, which = gz & 1;
  const int Dp = Dg * nb;
  const uint16_t* src = (which == 0 ? bases_k : bases_v) + (bases_shared ? 0 : (int64_t)b * Dp * rank) +
                        (int64_t)grp * Dg * rank;
  uint16_t* dst = bt + (((int64_t)b * 2 + which) * nb + grp) * (int64_t)rank * Dg;
  __shared__ uint16_t tile[32][256 + 2];
  // thread: row t / 8, 8-column pieces t % 8, t % 8 + 8, ..
  const int r = threadIdx.x >> 3;
  for (int c8 = threadIdx.x & 7; c8 < rank / 8; c8 += 8) {
    Op8 v;
    v.u = *reinterpret_cast<const uint4*>(src + (int64_t)(d0 + r) * rank + c8 * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) tile[r][c8 * 8 + i] = v.h[i];
  }
  __syncthreads();
  // thread: dims 8 (t % 4) .. + 7 of columns t / 4, t / 4 + 64, ..
  const int d8 = (threadIdx.x & 3) * 8;
  for (int c = threadIdx.x >> 2; c < rank; c += 64) {
    Op8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v.h[i] = tile[d8 + i][c];
    *reinterpret_cast<uint4*>(dst + (int64_t)c * Dg + d0 + d8) = v.u;
  }
}

template <int RBH>
__global__ __launch_bounds__(kPfWaves * 64, 2) void k_prefill_project(
    const uint16_t* __restrict__ s_k, const uint16_t* __restrict__ s_v, const uint16_t* __restrict__ bt_all,
    uint16_t* __restrict__ coef_k, uint16_t* __restrict__ coef_v, int64_t n_rows, int hkv, int dh, int nb, int R,
    int64_t cap) {
  constexpr int RANK = RBH * 32;
  constexpr int NCB = RANK / 16;                  // 16-column blocks of the group
  constexpr int NSL = 2 * NCB / kPfWaves;         // slice loads per wave and step (= RBH)
  constexpr int NROW = 2 * kPfTiles;              // row loads per wave and step
  const int blk = blockIdx.x, gz = blockIdx.y, b = blockIdx.z;
  const int grp = gz >> 1, which = gz & 1;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int slot = lane & 15, kq = lane >> 4;
  const int Dp = hkv * dh, Dg = Dp / nb;
  const int ns = Dg / kPfStep;
  const uint16_t* S = (which == 0 ? s_k : s_v) + (int64_t)b * n_rows * Dp + (int64_t)grp * Dg;
  const uint16_t* Bt = bt_all + (((int64_t)b * 2 + which) * nb + grp) * (int64_t)RANK * Dg;
  uint16_t* C = (which == 0 ? coef_k : coef_v) + (int64_t)b * cap * R;

  // slice buffers [32-dim half][column][32 dims], the four 16-byte
  // quarters of a column's row XORed with (column / 2) % 4 so that the operand
  // reads of eight consecutive columns hit distinct banks
  // (three arrays: the loads that refill one then never hold up the reads of
  // another)
  __shared__ __align__(16) uint16_t bt0[2][RANK][32], bt1[2][RANK][32], bt2[2][RANK][32];

  const int64_t blk0 = (int64_t)blk * kPfRows;
  // the workgroup's rows as a buffer: rows past the prompt and steps past the
  // group lie out of its range and read as zero without a memory access, so
  // the loads need no branch (which would make the compiler wait for them)
  const int rows_here = (int)min<int64_t>(kPfRows, n_rows - blk0);
  const uint32_t nbytes = (uint32_t)((rows_here - 1) * Dp + Dg) * 2u;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(S + blk0 * Dp), (short)0, (int)nbytes, 0x00020000);
  uint32_t roff[kPfTiles];
#pragma unroll
  for (int i = 0; i < kPfTiles; ++i) {
    const int r = (w * kPfTiles + i) * 16 + slot;
    roff[i] = r < rows_here ? (uint32_t)(r * Dp + kq * 8) * 2u : 0x80000000u;
  }
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  auto load_rows = [&](int st, Op8 (&a)[kPfTiles][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kPfTiles; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t o = st < ns ? roff[i] + (uint32_t)(st * kPfStep + h * 32) * 2u : 0x80000000u;
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0);
        a[i][h].u = make_uint4(v.x, v.y, v.z, v.w);
      }
  };
  // slice st: 2 NCB wave loads of 16 columns x 32 dims shared out over the
  // waves (lane l: column l / 4, quarter (l % 4) ^ ((l / 8) % 4) -> LDS byte
  // 16 l); past the last step the last slice again, into a buffer no longer read
  // (a macro, the LDS destination through a plain local pointer: with the
  // array expression passed to the builtin directly the host pass drops the
  // kernel's launch stub)
#define S4R_PF_ISSUE_SLICE(BT, ST)                                                                             \
  do {                                                                                                       \
    const int st_ = min((ST), ns - 1);                                                                       \
    _Pragma("unroll") for (int u = 0; u < NSL; ++u) {                                                        \
      const int n_ = u * kPfWaves + w, h_ = n_ & 1, c_ = n_ >> 1;                                            \
      uint16_t* dst_ = &BT[h_][16 * c_][0];                                                                   \
      __builtin_amdgcn_global_load_lds(Bt + (int64_t)(16 * c_ + (lane >> 2)) * Dg + st_ * kPfStep + h_ * 32 + \
                                           (((lane & 3) ^ ((lane >> 3) & 3)) * 8),                           \
                                       dst_, 16, 0, 0);                                                      \
    }                                                                                                        \
  } while (0)

  floatx4 acc[kPfTiles][NCB];
#pragma unroll
  for (int i = 0; i < kPfTiles; ++i)
#pragma unroll
    for (int n = 0; n < NCB; ++n) acc[i][n] = floatx4{0.f, 0.f, 0.f, 0.f};

  // issue order per wave: slice 0 and rows 0, slice 1 and rows 1, then in step
  // st rows st + 2 and slice st + 2: at the top of a step only the next step's
  // loads may still be in flight.  The waits count loads, so no load may move
  // from one step's group to another's (the scheduling barriers)
  Op8 a0[kPfTiles][2], a1[kPfTiles][2], a2[kPfTiles][2];
  S4R_PF_ISSUE_SLICE(bt0, 0);
  load_rows(0, a0);
  __builtin_amdgcn_sched_barrier(0);
  S4R_PF_ISSUE_SLICE(bt1, 1);
  load_rows(1, a1);
  __builtin_amdgcn_sched_barrier(0);
  const int koff = (kq ^ ((slot >> 1) & 3)) * 8;
  auto step = [&](auto buf, auto last, int st, const Op8 (&a)[kPfTiles][2], Op8 (&next)[kPfTiles][2])
                  __attribute__((always_inline)) {
    constexpr int BUF = decltype(buf)::value;      // st % 3
    constexpr bool LAST = decltype(last)::value;   // one of the last steps: nothing more to request
    if constexpr (LAST)
      pf_wait_vmcnt<0>();
    else
      pf_wait_vmcnt<NROW + NSL>();
    lds_barrier();                                 // every wave's part of slice st, and slice st - 1 read
    if constexpr (!LAST) {
      load_rows(st + 2, next);
      if constexpr (BUF == 0)
        S4R_PF_ISSUE_SLICE(bt2, st + 2);
      else if constexpr (BUF == 1)
        S4R_PF_ISSUE_SLICE(bt0, st + 2);
      else
        S4R_PF_ISSUE_SLICE(bt1, st + 2);
      __builtin_amdgcn_sched_barrier(0);           // the requests go out before the products
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int n = 0; n < NCB; ++n) {
        Op8 bop;
        bop.u = *reinterpret_cast<const uint4*>(BUF == 0   ? &bt0[h][n * 16 + slot][koff]
                                                : BUF == 1 ? &bt1[h][n * 16 + slot][koff]
                                                           : &bt2[h][n * 16 + slot][koff]);
#pragma unroll
        for (int i = 0; i < kPfTiles; ++i) acc[i][n] = mfma16x16x32(bop, a[i][h], acc[i][n]);
      }
  };
  // three steps per iteration without a branch between them (at a branch the
  // compiler waits for every load), the last one or two after the loop
  constexpr std::integral_constant<int, 0> k0{};
  constexpr std::integral_constant<int, 1> k1{};
  constexpr std::integral_constant<int, 2> k2{};
  int st = 0;
  for (; st + 3 <= ns; st += 3) {
    step(k0, std::false_type(), st, a0, a2);
    step(k1, std::false_type(), st + 1, a1, a0);
    step(k2, std::false_type(), st + 2, a2, a1);
  }
  if (st < ns) step(k0, std::true_type(), st, a0, a2);
  if (st + 1 < ns) step(k1, std::true_type(), st + 1, a1, a0);
#undef S4R_PF_ISSUE_SLICE
  pf_wait_vmcnt<0>();                              // no load into LDS outlives the workgroup
  // D layout: lane (row slot, column group kq) holds columns 4 kq + v of block n
  const int c0 = grp * RANK;
#pragma unroll
  for (int i = 0; i < kPfTiles; ++i) {
    const int64_t r = blk0 + (w * kPfTiles + i) * 16 + slot;
    if (r < n_rows) {
      uint16_t* cp = C + (r >> 4) * (int64_t)(kTileTok * R) + (r & 15) * kBlkCol;
#pragma unroll
      for (int n = 0; n < NCB; ++n) {
        const int c = c0 + n * 16 + 4 * kq;
        *reinterpret_cast<uint2*>(cp + (c >> 5) * (kTileTok * kBlkCol) + (c & 31)) =
            make_uint2(pack_bf16x2(acc[i][n][0], acc[i][n][1]), pack_bf16x2(acc[i][n][2], acc[i][n][3]));
      }
    }
  }
}

template <int RBH>
static void launch_pf(const Problem& P, int64_t n_rows, const void* s_k, const void* s_v, const uint16_t* bt,
                      void* coef_k, void* coef_v, hipStream_t st) {
  dim3 grid((unsigned)((n_rows + kPfRows - 1) / kPfRows), 2 * P.nb, P.B);
  hipLaunchKernelGGL(k_prefill_project<RBH>, grid, dim3(kPfWaves * 64), 0, st, (const uint16_t*)s_k,
                     (const uint16_t*)s_v, bt, (uint16_t*)coef_k, (uint16_t*)coef_v, n_rows, P.hkv, P.dh, P.nb, P.R,
                     P.cap);
}

size_t prefill_ws_bytes(const Problem& P) { return (size_t)P.B * 2 * P.hkv * P.dh * P.rank * 2; }

hipError_t launch_prefill_project(const Problem& P, int64_t n_rows, const void* s_k, const void* s_v,
                                  const void* bases_k, const void* bases_v, void* coef_k, void* coef_v, void* ws,
                                  hipStream_t st) {
  uint16_t* bt = (uint16_t*)ws;
  const int Dg = P.hkv * P.dh / P.nb;
  hipLaunchKernelGGL(k_transpose_bases, dim3(Dg / 32, 2 * P.nb, P.B), dim3(256), 0, st, (const uint16_t*)bases_k,
                     (const uint16_t*)bases_v, bt, Dg, P.nb, P.rank, P.bases_shared);
  switch (P.rank / 32) {
    case 1: launch_pf<1>(P, n_rows, s_k, s_v, bt, coef_k, coef_v, st); break;
    case 2: launch_pf<2>(P, n_rows, s_k, s_v, bt, coef_k, coef_v, st); break;
    case 3: launch_pf<3>(P, n_rows, s_k, s_v, bt, coef_k, coef_v, st); break;
    case 4: launch_pf<4>(P, n_rows, s_k, s_v, bt, coef_k, coef_v, st); break;
    case 5: launch_pf<5>(P, n_rows, s_k, s_v, bt, coef_k, coef_v, st); break;
    case 6: launch_pf<6>(P, n_rows, s_k, s_v, bt, coef_k, coef_v, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace s4r
