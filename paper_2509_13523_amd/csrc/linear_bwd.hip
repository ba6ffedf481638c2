// Gradients of a projection y = x W^T of an AERIS transformer layer (paper, Model Architecture
// section: the projections of queries, keys and values, the output projection and the SwiGLU
// feed-forward part; training runs the backward pass of each): dx = dy W and dW = dy^T x;
// argument contracts in include/aeris_layer_ops.h.
//
// dx is the forward GEMM kernel on the transposed weight (W^T [C, F], written by the kernel that also
// adds up dW), so both of its operands are contiguous along the contraction again.
//
// dW contracts over the token rows, along which neither operand is contiguous.  One workgroup
// owns a tile of dW for a range of rows; per step 64 rows of dy (the tile's features) and of x
// (its channels) go global -> LDS directly as [64][128] or [64][64] sub-tiles in the swizzled
// chunk layout of the attention kernels, and both MFMA operands are fetched with transposing
// reads (ds_read_b64_tr_b16), the token index landing in the registers.  The rows of the whole
// problem are split over several workgroups per tile; each writes its partial tile, and a second
// kernel adds the partials in a fixed order (no atomics: the result does not depend on the
// schedule).  Rows past the end in the last step are cleared, in the LDS or in the operands, before use.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "aeris_layer_ops.h"
#include "aeris_probe.h"
#include "aeris_winattn.h"
#include "projection_gemm.hpp"
#include "winattn_common.hpp"
#include "winattn_launch.hpp"

namespace aeris {
namespace {

constexpr int kTM = 64;                  // token rows per step

// FW x CW waves, each with FB x CB blocks of 32 x 32; STAGES steps in the LDS at a time.
template <int FW_, int CW_, int FB_, int CB_, int STAGES_, int PER_CU_>
struct WgradShape {
  static constexpr int FW = FW_, CW = CW_, FB = FB_, CB = CB_, kStages = STAGES_;
  static constexpr int kPerCu = PER_CU_;                 // workgroups a CU holds
  // Long sums in two levels: after kRun steps the accumulators are added to a second set and
  // start again, which keeps the rounding error of a workgroup that walks many rows at that of
  // one which walks 1024.  The largest shape has no registers for it and gets its rows split.
  static constexpr int kRun = FB_ * CB_ <= 4 ? 16 : 0;
  static constexpr int kWaves = FW * CW;
  static constexpr int kTF = FW * FB * 32;               // features per workgroup tile
  static constexpr int kTC = CW * CB * 32;               // channels per workgroup tile
  static constexpr int kWidth = kTF % 128 == 0 && kTC % 128 == 0 ? 128 : 64;   // columns of a sub-tile
  using Sub = Tile<kWidth, kWaves>;
  static constexpr int kSubBytes = kTM * kWidth * 2;
  static constexpr int kFSubs = kTF / kWidth, kCSubs = kTC / kWidth;
  static constexpr int kStageBytes = (kFSubs + kCSubs) * kSubBytes;   // dy sub-tiles, then x sub-tiles
  static constexpr int kRowsPerInst = 512 / kWidth;      // rows one copy instruction of a wave moves
  static constexpr int kPiecesPerSub = kTM / kRowsPerInst / kWaves;   // per wave
  static constexpr int kPieces = (kFSubs + kCSubs) * kPiecesPerSub;   // copies of a wave per step
  static_assert(kPiecesPerSub * kRowsPerInst * kWaves == kTM, "waves share a sub-tile evenly");
};
using WgradLarge = WgradShape<2, 4, 4, 2, 2, 1>;    // 256 x 256, eight waves, 128 KB
using WgradMedium = WgradShape<2, 2, 2, 2, 2, 2>;   // 128 x 128, four waves, 64 KB
using WgradSmall = WgradShape<2, 2, 1, 1, 3, 3>;    // 64 x 64, four waves, 48 KB

struct WgradParams {
  const bf16_t* dy;            // [M, F]
  const bf16_t* x;             // [M, C]
  float* out;                  // [splits][F, C]
  int F, C;
  int f_tiles, c_tiles;
  int splits;
  int steps_per_split, steps_total;      // steps of kTM rows
  int tail;                              // rows of the last step if it is not whole, else 0
};

// Workgroup id -> (split, feature tile, channel tile).  Work items are listed by row range, then
// by bands of four feature tiles.  Consecutive workgroup ids go to the eight XCDs in turn; pieces
// of the list as long as the workgroups an XCD runs at a time go to the XCDs in turn, so that
// those share 64-row pieces of dy and x through its L2 (four feature tiles by eight channel tiles
// where there are that many) and walk the rows together; the items left over, fewer than one
// piece per XCD, are shared out evenly.  No idle workgroups.
__device__ __forceinline__ void wgrad_tile(const WgradParams& p, int piece, int& split, int& ft,
                                           int& ct) {
  const int tiles = p.f_tiles * p.c_tiles, total = p.splits * tiles;
  const int whole = total / (8 * piece) * (8 * piece);
  const int xcd = blockIdx.x & 7;
  int item;
  if ((int)blockIdx.x < whole) {
    const int slot = blockIdx.x >> 3;
    item = (slot / piece * 8 + xcd) * piece + slot % piece;
  } else {
    const int left = total - whole, share = left >> 3, extra = left & 7;
    item = whole + xcd * share + (xcd < extra ? xcd : extra) + (((int)blockIdx.x - whole) >> 3);
  }
  split = item / tiles;
  const int t = item - split * tiles;
  const int band = t / (4 * p.c_tiles), r = t - band * 4 * p.c_tiles;
  const int height = p.f_tiles - 4 * band < 4 ? p.f_tiles - 4 * band : 4;
  ct = r / height;
  ft = 4 * band + r - ct * height;
}

// The two smaller shapes.  Bound by the latency of a step (copies, barrier, first operand reads), which the
// CU's other workgroups cover in part.  Against a loop with offsets worked out per step and the compiler's
// order, us: 20011 rows 768 -> 2304 82.1 -> 76.6, 20000 x 2048 -> 2048 167.9 -> 158.5, 2000 x 1024 -> 1024
// 14.0 -> 11.6, 1728 x 128 -> 1024 10.4 -> 9.6.
template <class S>
__global__ __launch_bounds__(S::kWaves * 64, S::kWaves * S::kPerCu / 4) void linear_wgrad_kernel(
    WgradParams p) {
  using Sub = typename S::Sub;
  constexpr int FB = S::FB, CB = S::CB, kP = S::kPieces;
  extern __shared__ __align__(16) unsigned char smem[];
  int split, ft, ct;
  wgrad_tile(p, 32 * S::kPerCu, split, ft, ct);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wf = wave / S::CW, wc = wave % S::CW;
  const int li = lane & 31, g = lane >> 5;
  const int f0 = ft * S::kTF, c0 = ct * S::kTC;
  const int s0 = split * p.steps_per_split;
  const int s1 = s0 + p.steps_per_split < p.steps_total ? s0 + p.steps_per_split : p.steps_total;

  // ---- copies: piece i of wave w moves kRowsPerInst rows of sub-tile i / kPiecesPerSub.  Lane:
  // row + lane / chunks, LDS chunk position lane % chunks, which holds source chunk
  // position ^ swz(row).  Columns past the end of a ragged last tile are clamped into the row
  // (their products are never stored), rows past the end of the last step to its last row.
  constexpr int kChunks = S::kWidth / 8;
  auto piece_row = [&](int i) __attribute__((always_inline)) {
    return S::kRowsPerInst * (wave + S::kWaves * (i % S::kPiecesPerSub)) + lane / kChunks;
  };
  uint32_t voff[kP];
#pragma unroll
  for (int i = 0; i < kP; ++i) {
    const int t = i / S::kPiecesPerSub;
    const int r = piece_row(i);
    const int chunk = (lane % kChunks) ^ Sub::swz(r);
    const bool is_dy = t < S::kFSubs;
    const int ld = is_dy ? p.F : p.C;
    int col = (is_dy ? f0 + S::kWidth * t : c0 + S::kWidth * (t - S::kFSubs)) + 8 * chunk;
    col = col < ld ? col : ld - 8;
    voff[i] = (uint32_t)(((long long)r * ld + col) * 2);
  }
  const uint32_t lds0 = lds_address(smem);
  // rows of dy and x of the step whose copies come next
  const unsigned long long dy_step = (unsigned long long)kTM * 2 * p.F;
  const unsigned long long x_step = (unsigned long long)kTM * 2 * p.C;
  unsigned long long dy_at = reinterpret_cast<unsigned long long>(p.dy) + s0 * dy_step;
  unsigned long long x_at = reinterpret_cast<unsigned long long>(p.x) + s0 * x_step;
  auto copy_piece = [&](int i, uint32_t stage, uint32_t enable) __attribute__((always_inline)) {
    const int t = i / S::kPiecesPerSub;
    async_copy16_off(voff[i], t < S::kFSubs ? dy_at : x_at,
                     stage + (uint32_t)(t * S::kSubBytes +
                                        ((wave + S::kWaves * (i % S::kPiecesPerSub)) << 10)),
                     enable);
  };

  // before the copies of step `step`: if rows are missing there, its (last) copies stop at the last row
  auto clamp_rows = [&](int step) __attribute__((always_inline)) {
    if (p.tail == 0 || step != p.steps_total - 1) return;
#pragma unroll
    for (int i = 0; i < kP; ++i) {
      const int past = piece_row(i) - (p.tail - 1);
      voff[i] -= past > 0 ? (uint32_t)past * (uint32_t)((i / S::kPiecesPerSub < S::kFSubs ? p.F : p.C) * 2) : 0u;
    }
  };

  // ---- transposing operand reads: per lane two addresses per 32-column block (rows 4g..4g+3
  // and 8+4g..8+4g+3 of a 16-row group; both operands use the same row order)
  uint32_t ta[FB][2], tb[CB][2];
  {
    const int j = lane & 15, blk = lane >> 4;
    // block of 32 columns starting at `col` of the operand whose first sub-tile is `first`
    auto address = [&](int first, int col, int h) __attribute__((always_inline)) {
      const int r = 8 * h + 4 * (blk >> 1) + (j >> 2);
      const int c = (col % S::kWidth) / 8 + 2 * (blk & 1) + ((j & 3) >> 1);
      return lds0 + (first + col / S::kWidth) * S::kSubBytes + Sub::chunk_offset(r, c) + (j & 1) * 8;
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int a = 0; a < FB; ++a) ta[a][h] = address(0, (wf * FB + a) * 32, h);
#pragma unroll
      for (int b = 0; b < CB; ++b) tb[b][h] = address(S::kFSubs, (wc * CB + b) * 32, h);
    }
  }

  f32x16 acc[FB][CB];
#pragma unroll
  for (int a = 0; a < FB; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  f32x16 sum[S::kRun ? FB : 1][S::kRun ? CB : 1];
  auto add_run = [&]() __attribute__((always_inline)) {
    if constexpr (S::kRun != 0) {
#pragma unroll
      for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            sum[a][b][i] += acc[a][b][i];
            acc[a][b][i] = 0.f;
          }
    }
  };
  if constexpr (S::kRun != 0) {
#pragma unroll
    for (int a = 0; a < FB; ++a)
#pragma unroll
      for (int b = 0; b < CB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[a][b][i] = 0.f;
  }

#pragma unroll
  for (int st = 0; st < S::kStages - 1; ++st) {
    if (s0 + st < s1) clamp_rows(s0 + st);
#pragma unroll
    for (int i = 0; i < kP; ++i) copy_piece(i, lds0 + st * S::kStageBytes, s0 + st < s1);
    dy_at += dy_step;
    x_at += x_step;
  }

  bf16x8 ao[2][FB], bo[2][CB];
  auto fetch_a = [&](int set, int kk, uint32_t from) __attribute__((always_inline)) {
    const uint32_t off = from + kk * (16 * S::kWidth * 2);
#pragma unroll
    for (int a = 0; a < FB; ++a) ao[set][a] = Sub::read_tr(ta[a][0] + off, ta[a][1] + off);
  };
  auto fetch_b = [&](int set, int kk, uint32_t from) __attribute__((always_inline)) {
    const uint32_t off = from + kk * (16 * S::kWidth * 2);
#pragma unroll
    for (int b = 0; b < CB; ++b) bo[set][b] = Sub::read_tr(tb[b][0] + off, tb[b][1] + off);
  };

  // The copies of a last step with rows missing are issued kStages - 1 steps ahead of it, and only from
  // there on do steps look for it.
  const int plain_end = p.tail && s1 == p.steps_total ? s1 - S::kStages : s1;
  // One step, in stage `slot`: LDS offsets are immediates, and products, reads and copies keep this order.
  auto run_step = [&](auto slot, int ks) __attribute__((always_inline)) {
    constexpr int kSlot = decltype(slot)::value;
    constexpr uint32_t kHere = kSlot * S::kStageBytes;
    constexpr uint32_t kFill = (kSlot + S::kStages - 1) % S::kStages * S::kStageBytes;
    // this stage's copies are the oldest in flight; those of the kStages - 2 steps behind it, if
    // there are that many, may stay in flight
    if (S::kStages > 2 && ks + S::kStages - 2 < s1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S::kStages - 2) * kP) : "memory");
    else wait_async_loads();
    __syncthreads();               // this stage has landed; every reader of the one filled next is done
    const int next = ks + S::kStages - 1;
    const uint32_t more = next < s1;
    if (ks >= plain_end) {
      if (p.tail && ks == p.steps_total - 1) {           // clear the rows past the end, once
        const int clear = (kTM - p.tail) * kChunks;      // 16-byte chunks per sub-tile
        for (int t = 0; t < S::kFSubs + S::kCSubs; ++t)
          for (int i = tid; i < clear; i += S::kWaves * 64)
            *reinterpret_cast<u32x4*>(smem + kHere + t * S::kSubBytes +
                                      (p.tail * kChunks + i) * 16) = u32x4{0, 0, 0, 0};
        __syncthreads();
      }
      if (more) clamp_rows(next);
    }
    fetch_a(0, 0, kHere);
    fetch_b(0, 0, kHere);
    sched_fence();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int q = 0; q < FB * CB; ++q) {
        const int a = q / CB, b = q % CB;
        acc[a][b] = mfma32(ao[kk & 1][a], bo[kk & 1][b], acc[a][b]);
        if (kk < 3 && q == 0) fetch_a((kk + 1) & 1, kk + 1, kHere);
        if (kk < 3 && q == (FB * CB == 1 ? 0 : 1)) fetch_b((kk + 1) & 1, kk + 1, kHere);
        // the copies of a later stage ride in the first half of the step, spread evenly
        constexpr int kHalf = 2 * FB * CB;
        const int n = kk * FB * CB + q;
        if (n < kHalf) {
#pragma unroll
          for (int i = n * kP / kHalf; i < (n + 1) * kP / kHalf; ++i) copy_piece(i, lds0 + kFill, more);
        }
        sched_fence();
      }
    }
    if (S::kRun != 0 && ((ks - s0) & (S::kRun - 1)) == S::kRun - 1) add_run();
    dy_at += dy_step;
    x_at += x_step;
  };
  static_assert(S::kStages == 2 || S::kStages == 3);
  for (int ks = s0;;) {
    run_step(Const<0>{}, ks);
    if (++ks == s1) break;
    run_step(Const<1>{}, ks);
    if (++ks == s1) break;
    if constexpr (S::kStages == 3) {
      run_step(Const<2>{}, ks);
      if (++ks == s1) break;
    }
  }

  add_run();
  // ---- partial tile: a lane owns one channel column, a register one feature row
  float* out = p.out + (long long)split * p.F * p.C;
#pragma unroll
  for (int a = 0; a < FB; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int c = c0 + (wc * CB + b) * 32 + li;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int f = f0 + (wf * FB + a) * 32 + acc_row(e, g);
        if (f < p.F && c < p.C) out[(long long)f * p.C + c] = S::kRun ? sum[a][b][e] : acc[a][b][e];
      }
    }
}

// The same for the 256 x 256 shape, whose two waves of a SIMD take turns as in projection_gemm_kernel:
// a step is two halves of 32 rows and 16 products, and waves 4-7 run one barrier behind waves 0-3, so
// that one multiplies while the other fetches its operands and issues copies.  A half of a stage is
// copied over as soon as both waves have its operands in registers, three halves ahead of its use.
// Bound by the board's power cap.  172800 rows, us, all waves together / in turns, one session: 2048 -> 2048
// 1390 / 1251, 2048 -> 6144 3655 / 3461, 5504 -> 2048 3572 / 3325.
//
// The 32 workgroups of an XCD that walk the same rows share them through its L2 only while they stay
// together.  A wave that waits for its copies is held when it leads (they come from memory) and not when it
// follows (from the L2), but copies issued three halves ahead are hardly ever waited for, and in a long range the
// workgroups drift apart (4,147,200 rows, 2048 -> 6144, 12 ranges of 5400 steps: 732 GB fetched into the L2s
// where 166 had been, 81.5 -> 93.7 ms).  So long ranges wait for copies issued one half earlier (kNear), and the
// longest also for all of them at every 64th step (kHeld).  us, all waves together / kFar / kNear / kHeld:
//   rows x channels -> features   steps of a range
//   130000 x 2048 -> 2048           64               1062 /   948 /   980 /   992
//   172800 x 2048 -> 2048           85               1380 /  1198 /  1226 /  1265
//   100000 x 2048 -> 6144          131               2166 /  1980 /  2002 /  2058
//   300000 x 2048 -> 2048          147               2231 /  1948 /  1980 /  2040
//   400000 x 2048 -> 2048          196               2934 /  2559 /  2578 /  2679
//   172800 x 5504 -> 2048          225               3473 /  3194 /  3166 /  3271
//   230000 x 2048 -> 6144          300               4694 /  4435 /  4362 /  4464
//   172800 x 2048 -> 11008         338               6452 /  6189 /  6072 /  6069
//   400000 x 2048 -> 6144          521               8030 /  7819 /  7503 /  7621
//   691200 x 2048 -> 6144          900              13619 / 13852 / 12902 / 13155
//   1036800 x 5504 -> 2048        1350              20702 / 21344 / 20424 / 20203
//   1036800 x 2048 -> 11008       2025              37508 / 40231 / 38587 / 37728
//   4147200 x 2048 -> 6144        5400              81497 / 93697 / 84310 / 81022
enum class Pace { kFar, kNear, kHeld };
constexpr int kNearFromSteps = 211, kHeldFromSteps = 1200;

template <Pace kPace>
__global__ __launch_bounds__(512, 2) void linear_wgrad_large_kernel(WgradParams p) {
  using S = WgradLarge;
  using Sub = S::Sub;
  constexpr int FB = S::FB, CB = S::CB, kP = S::kPieces, kSubs = S::kFSubs + S::kCSubs;
  static_assert(S::kPiecesPerSub == 2 && S::kStages == 2 && S::kRun == 0);
  extern __shared__ __align__(16) unsigned char smem[];
  int split, ft, ct;
  wgrad_tile(p, 32, split, ft, ct);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wf = wave / S::CW, wc = wave % S::CW;
  const int li = lane & 31, g = lane >> 5;
  const int f0 = ft * S::kTF, c0 = ct * S::kTC;
  const int s0 = split * p.steps_per_split;
  const int s1 = s0 + p.steps_per_split < p.steps_total ? s0 + p.steps_per_split : p.steps_total;

  // ---- copies, as above; piece 2 t + h of a wave: four rows of half h of sub-tile t
  constexpr int kChunks = S::kWidth / 8;
  auto piece_row = [&](int i) __attribute__((always_inline)) {
    return S::kRowsPerInst * (wave + S::kWaves * (i & 1)) + lane / kChunks;
  };
  uint32_t voff[kP];
#pragma unroll
  for (int i = 0; i < kP; ++i) {
    const int t = i >> 1, r = piece_row(i), chunk = (lane % kChunks) ^ Sub::swz(r);
    const bool is_dy = t < S::kFSubs;
    const int ld = is_dy ? p.F : p.C;
    int col = (is_dy ? f0 + S::kWidth * t : c0 + S::kWidth * (t - S::kFSubs)) + 8 * chunk;
    col = col < ld ? col : ld - 8;
    voff[i] = (uint32_t)(((long long)r * ld + col) * 2);
  }
  const uint32_t lds0 = lds_address(smem);
  const unsigned long long dy_step = (unsigned long long)kTM * 2 * p.F;
  const unsigned long long x_step = (unsigned long long)kTM * 2 * p.C;
  const unsigned long long dy0 = reinterpret_cast<unsigned long long>(p.dy), x0 = reinterpret_cast<unsigned long long>(p.x);
  auto copy_rows = [&](int h, uint32_t stage, unsigned long long dy_at, unsigned long long x_at)
      __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < kSubs; ++t)
      async_copy16_at(voff[2 * t + h], t < S::kFSubs ? dy_at : x_at,
                      lds0 + stage + (uint32_t)(t * S::kSubBytes + ((wave + S::kWaves * h) << 10)));
  };
  auto copy_half = [&](int h, uint32_t stage, int step) __attribute__((always_inline)) {
    if (p.tail != 0 && step == p.steps_total - 1) {        // the last copies of all stop at the last row
#pragma unroll
      for (int t = 0; t < kSubs; ++t) {
        const int past = piece_row(2 * t + h) - (p.tail - 1);
        voff[2 * t + h] -= past > 0 ? (uint32_t)past * (uint32_t)((t < S::kFSubs ? p.F : p.C) * 2) : 0u;
      }
    }
    copy_rows(h, stage, dy0 + step * dy_step, x0 + step * x_step);
  };

  // ---- transposing operand reads, as above
  uint32_t ta[FB][2], tb[CB][2];
  {
    const int j = lane & 15, blk = lane >> 4;
    auto address = [&](int first, int col, int h) __attribute__((always_inline)) {
      const int r = 8 * h + 4 * (blk >> 1) + (j >> 2);
      const int c = (col % S::kWidth) / 8 + 2 * (blk & 1) + ((j & 3) >> 1);
      return lds0 + (first + col / S::kWidth) * S::kSubBytes + Sub::chunk_offset(r, c) + (j & 1) * 8;
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int a = 0; a < FB; ++a) ta[a][h] = address(0, (wf * FB + a) * 32, h);
#pragma unroll
      for (int b = 0; b < CB; ++b) tb[b][h] = address(S::kFSubs, (wc * CB + b) * 32, h);
    }
  }

  f32x16 acc[FB][CB];
#pragma unroll
  for (int a = 0; a < FB; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  bf16x8 ao[2][FB], bo[2][CB];
  auto landed = [&](auto behind) __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(behind)::value) : "memory");
  };
  auto fetch = [&](int h, uint32_t here) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const uint32_t off = here + (2 * h + kk) * (16 * S::kWidth * 2);
#pragma unroll
      for (int a = 0; a < FB; ++a) ao[kk][a] = Sub::read_tr(ta[a][0] + off, ta[a][1] + off);
#pragma unroll
      for (int b = 0; b < CB; ++b) bo[kk][b] = Sub::read_tr(tb[b][0] + off, tb[b][1] + off);
    }
  };
  // rows past the end, which hold copies of the last row, are cleared in the operands of both sides
  auto clear_past_end = [&](int h) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int row0 = (2 * h + kk) * 16 + 4 * g;          // element e: row row0 + 8 (e / 4) + e % 4
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool keep = row0 + 8 * (e >> 2) + (e & 3) < p.tail;
#pragma unroll
        for (int a = 0; a < FB; ++a) ao[kk][a][e] = keep ? ao[kk][a][e] : (bf16_t)0.f;
#pragma unroll
        for (int b = 0; b < CB; ++b) bo[kk][b][e] = keep ? bo[kk][b][e] : (bf16_t)0.f;
      }
    }
  };
  auto products = [&]() __attribute__((always_inline)) {
    lds_barrier();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[a][b] = mfma32(ao[kk][a], bo[kk][b], acc[a][b]);
    __builtin_amdgcn_s_setprio(0);
    lds_barrier();
  };

  copy_half(0, 0, s0);
  copy_half(1, 0, s0);
  if (s0 + 1 < s1) {
    copy_half(0, S::kStageBytes, s0 + 1);
    landed(Const<8>{});
  } else {
    landed(Const<4>{});
  }
  lds_barrier();
  if (wf == 1) lds_barrier();
  uint32_t here = 0;
  int ks = s0;
  // steps that copy whole steps only; those look for no last one, and their addresses need no products
  const int plain_end = p.tail != 0 && s1 == p.steps_total ? s1 - 1 : s1;
  unsigned long long dy_at = dy0 + (s0 + 1) * dy_step, x_at = x0 + (s0 + 1) * x_step;   // of the next step
  constexpr int kBehind = kPace == Pace::kFar ? 8 : 4;      // copies that may be on their way
  for (; ks + 2 < plain_end; ++ks, here = S::kStageBytes - here) {
    fetch(0, here);
    copy_rows(1, S::kStageBytes - here, dy_at, x_at);
    if (kPace == Pace::kHeld && ((ks - s0) & 63) == 63) landed(Const<0>{});
    else landed(Const<kBehind>{});
    products();
    dy_at += dy_step;
    x_at += x_step;
    fetch(1, here);
    copy_rows(0, here, dy_at, x_at);
    landed(Const<kBehind>{});
    products();
  }
  for (; ks < s1; ++ks, here = S::kStageBytes - here) {
    const bool clear = p.tail != 0 && ks == p.steps_total - 1, more = ks + 1 < s1;
    fetch(0, here);
    if (more) {
      copy_half(1, S::kStageBytes - here, ks + 1);
      landed(Const<8>{});
    } else {
      landed(Const<0>{});
    }
    if (clear) clear_past_end(0);
    products();
    fetch(1, here);
    if (ks + 2 < s1) {
      copy_half(0, here, ks + 2);
      landed(Const<8>{});
    } else if (more) {
      landed(Const<4>{});
    }
    if (clear) clear_past_end(1);
    products();
  }
  if (wf == 0) lds_barrier();

  // ---- partial tile: a lane owns one channel column, a register one feature row
  float* out = p.out + (long long)split * p.F * p.C;
#pragma unroll
  for (int a = 0; a < FB; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int c = c0 + (wc * CB + b) * 32 + li;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int f = f0 + (wf * FB + a) * 32 + acc_row(e, g);
        if (f < p.F && c < p.C) out[(long long)f * p.C + c] = acc[a][b][e];
      }
    }
}

// dW = sum of the partial tiles, in the order of the splits.  n4: number of 4-float groups of dW.
// kInFlight loads of a thread at a time: eight where few threads have to cover the latency (65536 x 4
// bytes, 48 ranges: 30 us with one, 23 with eight); one where a full grid does and more streams only
// spread over more pages (2048 x 2048, 32 ranges: 123 us with eight, 101 with one).  Workgroup `block` of
// `blocks`.
template <int kInFlight>
__device__ __forceinline__ void wgrad_reduce(const float* __restrict__ part, long long n4, int splits,
                                             float* __restrict__ dw, unsigned block, unsigned blocks) {
  const long long stride = (long long)blocks * 256;
  for (long long i = (long long)block * 256 + threadIdx.x; i < n4; i += stride) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll kInFlight
    for (int k = 0; k < splits; ++k) {
      const f32x4 v = reinterpret_cast<const f32x4*>(part)[(long long)k * n4 + i];
      s[0] += v[0]; s[1] += v[1]; s[2] += v[2]; s[3] += v[3];
    }
    reinterpret_cast<f32x4*>(dw)[i] = s;
  }
}

// wt [C, F] = w [F, C]^T, bf16: 64 x 64 tiles through the LDS, 16 bytes per lane and access on
// both sides (C and F are multiples of 64, so every tile is whole).  Bound by the latency of one
// load and one store: two of each per thread, all in flight together.  The pitch of 66 elements
// puts the eight scattered 2-byte writes of a lane and its neighbours into different banks.
__device__ __forceinline__ void transpose_weight(const bf16_t* __restrict__ w, int F, int C,
                                                 bf16_t* __restrict__ wt, unsigned block) {
  constexpr int kPitch = 66;
  typedef uint32_t __attribute__((may_alias)) pair_t;          // two features, read as one word
  __shared__ __align__(4) unsigned short tile[64 * kPitch];    // [channel][feature]
  const unsigned c_tiles = (unsigned)C / 64;
  const int f0 = (int)(block / c_tiles) * 64, c0 = (int)(block % c_tiles) * 64;
  const int row = threadIdx.x >> 3, chunk = threadIdx.x & 7;   // rows row, row + 32
  u32x4 v[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    v[i] = *reinterpret_cast<const u32x4*>(w + (long long)(f0 + row + 32 * i) * C + c0 + 8 * chunk);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      tile[(8 * chunk + e) * kPitch + row + 32 * i] = (unsigned short)(v[i][e >> 1] >> (16 * (e & 1)));
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const pair_t* src = reinterpret_cast<const pair_t*>(tile + (row + 32 * i) * kPitch + 8 * chunk);
    *reinterpret_cast<u32x4*>(wt + (long long)(c0 + row + 32 * i) * F + f0 + 8 * chunk) =
        u32x4{src[0], src[1], src[2], src[3]};
  }
}

// Between the two products: the transposed weight that dx multiplies with, in the first transpose_blocks
// workgroups, and the sum of dW's partial tiles in the others, side by side in one launch instead of two: 2.5 to
// 5 us less on the GPU and 3 us on the host per call (20,011 rows, 768 -> 2304: 161.6 -> 155.7 us; with
// norm_fold_kernel a layer of 1728 rows x 128, bound by the host at 40 launches, 258 -> 237 us at 34).
template <int kInFlight>
__global__ __launch_bounds__(256) void between_kernel(const bf16_t* __restrict__ w, int F, int C,
                                                      bf16_t* __restrict__ wt, unsigned transpose_blocks,
                                                      const float* __restrict__ part, long long n4, int splits,
                                                      float* __restrict__ dw) {
  if (blockIdx.x < transpose_blocks) transpose_weight(w, F, C, wt, blockIdx.x);
  else wgrad_reduce<kInFlight>(part, n4, splits, dw, blockIdx.x - transpose_blocks, gridDim.x - transpose_blocks);
}

size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }
bool bad16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) != 0; }

enum class WgradTile { kLarge, kMedium, kSmall };
struct WgradPlan {
  WgradTile tile;
  int steps_total, steps_per_split, splits;
  int most;      // partial tiles the workspace holds; with one, dW itself is written
};

// Microseconds from the first workgroup to the last partial sum.  A CU that holds kPerCu of its n
// workgroups at a time takes step_us[kPerCu] per step of a full set and step_us[m] for a last set
// of m; the partial tiles cost a second launch and 0.25 us per MB written and read.
template <class S>
double wgrad_time(int splits, int per, int32_t channels, int32_t features, double fixed,
                  const double (&step_us)[4]) {
  const long long tiles = (long long)((features + S::kTF - 1) / S::kTF) * ((channels + S::kTC - 1) / S::kTC);
  const long long n = (tiles * splits + 255) / 256, sets = n / S::kPerCu, left = n % S::kPerCu;
  const double steps = (double)per * ((double)sets * step_us[S::kPerCu] + step_us[left]);
  const double sums = splits == 1 ? 0.0 : 3.0 + 0.25e-6 * ((double)splits * features * channels * 4.0);
  return steps + fixed * (double)(sets + (left != 0)) + sums;
}

// Row ranges of the largest tiles, 0 if there is no whole step: enough for about 2048 workgroups, at
// most 64 and no more than pieces of 16 steps give (the plan then makes them equally long: 17 steps
// are cut 9 + 8); among the next few counts the one whose units of 32 tiles (the
// workgroups an XCD runs at a time) share out to the eight XCDs most evenly.  Fixed by size alone:
// callers hold workspaces for this many partial tiles, and fewer ranges would be longer chains of
// additions, which this shape does not break up (23434 x 2112 -> 10560 in 6 ranges of 62 steps instead
// of 8 of 46: error of dW 2.9e-7 instead of 2.5e-7).
int large_ranges(int whole_steps, int32_t channels, int32_t features) {
  const int f_tiles = (features + WgradLarge::kTF - 1) / WgradLarge::kTF;
  const int c_tiles = (channels + WgradLarge::kTC - 1) / WgradLarge::kTC;
  const int unit_c = c_tiles >= 8 ? 8 : c_tiles >= 4 ? 4 : c_tiles >= 2 ? 2 : 1, unit_f = 32 / unit_c;
  const long long units_per_range =
      (long long)((f_tiles + unit_f - 1) / unit_f) * ((c_tiles + unit_c - 1) / unit_c);
  const long long tiles = (long long)f_tiles * c_tiles;
  const int want = (int)(2048 / tiles < 64 ? (2047 + tiles) / tiles : 64);
  int best = 0;
  double best_fill = -1.0;
  for (int target = want; target < want + 8 && target <= 64; ++target) {
    int per = (whole_steps + target - 1) / target;
    per = per < 16 ? 16 : per;
    const int ranges = (whole_steps + per - 1) / per;
    const long long units = ranges * units_per_range;
    const double fill = (double)units / (double)((units + 7) / 8 * 8);
    if (ranges > 0 && fill > best_fill + 1e-9) {
      best_fill = fill;
      best = ranges;
    }
  }
  return best;
}

// The plan that is estimated to end first.  Times per step measured over 1000 ... 172800 rows,
// 128 ... 5504 channels and 128 ... 11008 features; the 256 x 256 shape alone took (start to end, us)
// 43 / 44 / 98 / 159 / 117 / 79, with all its waves together, where this takes 12 / 22 / 80 / 86 / 72 / 55: 1000 x 1024 -> 1024,
// 4000 x 512 -> 1536, 8000 x 2048 -> 2048, 20011 x 768 -> 2304, 30000 x 1024 -> 1024,
// 100000 x 256 -> 768.  The smaller shapes take as many ranges as the largest has, or fewer: the
// workspace holds that many partial tiles (plan.most), and their chains of additions are broken up.
WgradPlan choose_wgrad(int64_t n_rows, int32_t channels, int32_t features) {
  WgradPlan best{};
  const int steps = (int)((n_rows + kTM - 1) / kTM);
  double best_time = 1e30;
  auto consider = [&](WgradTile tile, int want, auto time) {
    const int per = (steps + want - 1) / want;
    const int splits = (steps + per - 1) / per;
    const double t = time(splits, per);
    if (t >= best_time) return;
    best_time = t;
    best = WgradPlan{tile, steps, per, splits, best.most};
  };
  const int ranges = large_ranges((int)(n_rows / kTM), channels, features);
  best.most = ranges > 1 ? ranges : 1;
  if (ranges > 0)
    consider(WgradTile::kLarge, ranges, [&](int splits, int per) {
      return wgrad_time<WgradLarge>(splits, per, channels, features, 8.0, {0.0, 1.42, 0.0, 0.0});
    });
  for (int want = 1; want <= best.most && want <= steps; ++want) {
    consider(WgradTile::kMedium, want, [&](int splits, int per) {
      return wgrad_time<WgradMedium>(splits, per, channels, features, 5.0, {0.0, 0.72, 1.0, 0.0});
    });
    consider(WgradTile::kSmall, want, [&](int splits, int per) {
      return wgrad_time<WgradSmall>(splits, per, channels, features, 4.0, {0.0, 0.36, 0.44, 0.58});
    });
  }
  return best;
}

template <class S>
int launch_wgrad(WgradParams p, hipStream_t stream) {
  p.f_tiles = (p.F + S::kTF - 1) / S::kTF;
  p.c_tiles = (p.C + S::kTC - 1) / S::kTC;
  auto launch = [&](auto kernel) {
    return launch_kernel(kernel, dim3((unsigned)(p.splits * p.f_tiles * p.c_tiles)), dim3(S::kWaves * 64),
                         (size_t)S::kStages * S::kStageBytes, stream, p);
  };
  if constexpr (std::is_same<S, WgradLarge>::value) {
    auto launch_at = [&](auto pace) {
      constexpr auto kernel = linear_wgrad_large_kernel<decltype(pace)::value>;
      return allow_full_lds<kernel>() ? launch(kernel) : -1;
    };
    if (p.steps_per_split >= kHeldFromSteps) return launch_at(std::integral_constant<Pace, Pace::kHeld>{});
    if (p.steps_per_split >= kNearFromSteps) return launch_at(std::integral_constant<Pace, Pace::kNear>{});
    return launch_at(std::integral_constant<Pace, Pace::kFar>{});
  } else
    return allow_full_lds<linear_wgrad_kernel<S>>() ? launch(linear_wgrad_kernel<S>) : -1;
}

int check_linear_bwd(int64_t n_rows, int32_t channels, int32_t features) {
  if (n_rows <= 0 || channels <= 0 || features <= 0) return AERIS_ERR_INVALID_SHAPE;
  if (channels % 64 != 0 || features % 64 != 0) return AERIS_ERR_NOT_DIVISIBLE;
  if (n_rows / kTM >= (1LL << 31)) return AERIS_ERR_INVALID_SHAPE;
  // dx: the forward kernel with the roles of channels and features exchanged
  if (const int rc = projection_gemm_check(n_rows, n_rows, features, channels)) return rc;
  // dW: 32-bit byte offsets inside a 64-row step
  if ((long long)kTM * (features > channels ? features : channels) * 2 >= (1LL << 32))
    return AERIS_ERR_INVALID_SHAPE;
  return AERIS_OK;
}

}  // namespace
}  // namespace aeris

using namespace aeris;

// most: WgradPlan::most
static size_t workspace_bytes_of(int64_t n_rows, int32_t channels, int32_t out_features, int most) {
  // one partial tile is asked for where rows are left over a single row range, though dW itself is
  // written then: the size callers have known
  const bool none = n_rows < kTM || (most == 1 && n_rows % kTM == 0);
  return round256((size_t)out_features * channels * 2) +
         (none ? 0 : round256((size_t)most * out_features * channels * 4));
}

extern "C" size_t aeris_linear_bwd_workspace_bytes(int64_t n_rows, int32_t channels,
                                                   int32_t out_features) {
  if (check_linear_bwd(n_rows, channels, out_features) != AERIS_OK) return 0;
  return workspace_bytes_of(n_rows, channels, out_features, choose_wgrad(n_rows, channels, out_features).most);
}

extern "C" int aeris_linear_bwd_plan(int64_t n_rows, int32_t channels, int32_t out_features,
                                     int32_t* tile, int32_t* ranges, int32_t* steps) {
  if (!tile || !ranges || !steps) return AERIS_ERR_NULL_POINTER;
  if (const int rc = check_linear_bwd(n_rows, channels, out_features)) return rc;
  const WgradPlan plan = choose_wgrad(n_rows, channels, out_features);
  *tile = plan.tile == WgradTile::kLarge ? 256 : plan.tile == WgradTile::kMedium ? 128 : 64;
  *ranges = plan.splits;
  *steps = plan.steps_per_split;
  return AERIS_OK;
}

extern "C" int aeris_linear_bwd(const void* x, const void* weight, const void* dy, int64_t n_rows,
                                int32_t channels, int32_t out_features, void* dx, float* dweight,
                                void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!dy || !workspace || (!dx && !dweight) || (dx && !weight) || (dweight && !x))
    return AERIS_ERR_NULL_POINTER;
  if (const int rc = check_linear_bwd(n_rows, channels, out_features)) return rc;
  if (bad16(x) || bad16(weight) || bad16(dy) || bad16(dx) || bad16(dweight) || bad16(workspace))
    return AERIS_ERR_MISALIGNED;
  const WgradPlan plan = choose_wgrad(n_rows, channels, out_features);
  if (workspace_bytes < workspace_bytes_of(n_rows, channels, out_features, plan.most))
    return AERIS_ERR_WORKSPACE_TOO_SMALL;
  const hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(workspace);
  bf16_t* wt = reinterpret_cast<bf16_t*>(ws);
  float* part = reinterpret_cast<float*>(ws + round256((size_t)out_features * channels * 2));

  // dW's partial tiles; then the transposed weight and the sum of the tiles; then dx
  unsigned reduce_blocks = 0;
  int splits = 1;
  const long long n4 = (long long)out_features * channels / 4;
  if (dweight) {
    WgradParams p{};
    p.dy = static_cast<const bf16_t*>(dy);
    p.x = static_cast<const bf16_t*>(x);
    const bool direct = plan.splits == 1;
    p.out = direct ? dweight : part;
    p.F = out_features;
    p.C = channels;
    p.splits = splits = plan.splits;
    p.steps_per_split = plan.steps_per_split;
    p.steps_total = plan.steps_total;
    p.tail = (int)(n_rows % kTM);
    int rc = -1;
    switch (plan.tile) {
      case WgradTile::kLarge: rc = launch_wgrad<WgradLarge>(p, st); break;
      case WgradTile::kMedium: rc = launch_wgrad<WgradMedium>(p, st); break;
      case WgradTile::kSmall: rc = launch_wgrad<WgradSmall>(p, st); break;
    }
    if (rc != 0) return AERIS_ERR_HIP_LAUNCH;
    const long long blocks = (n4 + 255) / 256;
    if (!direct) reduce_blocks = (unsigned)(blocks < 4096 ? blocks : 4096);
  }
  const unsigned transpose_blocks = dx ? (unsigned)(channels / 64) * (unsigned)(out_features / 64) : 0;
  if (transpose_blocks + reduce_blocks != 0 &&
      launch_kernel(reduce_blocks < 4096 ? between_kernel<8> : between_kernel<1>,
                    dim3(transpose_blocks + reduce_blocks), dim3(256), 0, st,
                    static_cast<const bf16_t*>(weight), out_features, channels, wt, transpose_blocks,
                    static_cast<const float*>(part), n4, splits, dweight) != 0)
    return AERIS_ERR_HIP_LAUNCH;
  if (dx) {
    GemmParams p{};
    p.x = static_cast<const bf16_t*>(dy);
    p.w = wt;
    p.y = static_cast<bf16_t*>(dx);
    p.rows_per_sample = n_rows;
    p.n_samples = 1;
    p.K = out_features;
    p.F = channels;
    if (launch_projection_gemm(p, st) != 0) return AERIS_ERR_HIP_LAUNCH;
  }
  return AERIS_OK;
}
