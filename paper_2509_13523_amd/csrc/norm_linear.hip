// Input projections of an AERIS transformer layer with the pre-RMSNorm and the adaptive
// modulation folded in (paper, Model Architecture section: RMSNorm and the adaptive-layer-norm
// values precede the projection of queries, keys and values and the SwiGLU feed-forward part);
// argument contracts in include/aeris_layer_ops.h.
//
// The normalised, modulated row h_c = x_c r w_c (1 + gamma_bc) + beta_bc is never written:
//     y_f = sum_c h_c W_fc = r * sum_c x_c (W_fc w_c (1 + gamma_bc)) + sum_c beta_bc W_fc,
// so the projection is a plain bf16 GEMM of the raw rows x with a per-sample folded weight
//     Wf_b = W diag(w (1 + gamma_b))        (bf16, built by a small kernel per call)
// followed, in the epilogue, by the row's reciprocal RMS r (from a row pass over x) and a
// per-sample bias beta_b W^T.  The SwiGLU gate is a second epilogue: a workgroup's tile holds
// matching u and v columns, so g = silu(u) v is formed on the accumulators.
//
// GEMM kernels: 256 x 256 output tiles of eight wavefronts (128 x 128 of four or 64 x 64 of two where
// there are too few rows for that, see choose_gemm_tile), 64 channels per
// step, both operands K-contiguous ("NT").  Operand tiles go global -> LDS directly
// (global_load_lds_dwordx4), two stages or more, 16-byte chunks XOR-swizzled so that the
// row-major ds_read_b128 operand fetches are conflict free; v_mfma_f32_32x32x16_bf16 with the
// weight rows as the A operand and the token rows as the B operand, so that a lane owns one
// token row of the output: the row scale is a per-lane scalar.  Results are staged through the
// LDS and leave in 16-byte pieces, eight lanes per 128-byte row segment.
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

constexpr int kBK = 64;                  // channels per step
constexpr unsigned kCus = 256;           // of the chip
using Sub = Tile<64, 8>;                 // chunk swizzle of rows of 64 channels

// A workgroup tile of WM x WN wavefronts, each NB * 32 token rows x 64 features, and kStages
// operand stages (weight rows, then token rows) in the LDS.
template <int WM_, int WN_, int NB_, int STAGES_>
struct GemmShape {
  static constexpr int WM = WM_, WN = WN_, NB = NB_, kStages = STAGES_;
  static constexpr int kWaves = WM * WN;
  static constexpr int kBM = WM * NB * 32;             // token rows
  static constexpr int kBN = WN * 64;                  // weight rows (output features)
  static constexpr int kPartBytes = kBN * kBK * 2;     // weight rows of a stage
  static constexpr int kStageBytes = kPartBytes + kBM * kBK * 2;
  static constexpr int kSmem = kStages * kStageBytes;
  static constexpr int kStoreBlocks = NB < 2 ? NB : 2; // 32-row blocks a wave stages at a time
  static constexpr int kStoreBytes = kStoreBlocks * 32 * 128;   // ... in a region of this size
  static_assert(kWaves * kStoreBytes <= kStageBytes, "results are staged in one operand stage");
  // every wave issues four weight-row and four token-row copies of a stage
  static_assert(kBN == 32 * kWaves && kBM == 32 * kWaves && kWaves % 2 == 0);
};
using GemmLarge = GemmShape<2, 4, 4, 2>;   // 256 x 256, one workgroup per CU
using GemmMedium = GemmShape<2, 2, 2, 2>;  // 128 x 128, two workgroups per CU
using GemmSmall = GemmShape<2, 1, 1, 4>;   // 64 x 64, two workgroups per CU, three stages in flight

// Work item -> (token tile, feature tile); false if the item has no tile, nor has any later one of the
// same workgroup.  Items go to the XCDs in turn, as workgroup ids do.  Tiles are walked in
// groups of eight token tiles, feature tile by feature tile, so that the 32 tiles an XCD runs at a
// time are 8 token tiles x 4 feature tiles and every operand tile that arrives in that XCD's L2
// serves 4 or 8 workgroups.  Which token tiles an XCD owns: see interleave_tiles.
__device__ __forceinline__ bool gemm_tile(const GemmParams& p, int item, int& mt, int& nt) {
  const int per_group = 8 * p.n_tiles;
  int slot, m_tiles;
  if (p.interleave) {          // every eighth
    slot = item >> 3;
    m_tiles = (p.m_tiles + 7 - (item & 7)) >> 3;
    if (slot >= m_tiles * p.n_tiles) return false;
  } else {
    if (item >= p.m_tiles * p.n_tiles) return false;
    slot = xcd_contiguous(item, p.m_tiles * p.n_tiles);
    m_tiles = p.m_tiles;
  }
  const int group = slot / per_group, rem = slot - group * per_group;
  const int left = m_tiles - group * 8, gm = left < 8 ? left : 8;
  nt = rem / gm;
  mt = group * 8 + (rem - nt * gm);
  if (p.interleave) mt = mt * 8 + (item & 7);
  return true;
}

// Whether the XCDs take the token tiles in turn, or each a contiguous range of the list of all tiles.
// In turn is the faster one (time over that of ranges 0.92-1.03, mean 0.98, over 2000 ... 172800 rows,
// 192 ... 8192 channels, 192 ... 6144 features; never above 1.02 of that of groups padded to eight
// token tiles, whose idle workgroups unbalance the shader engines: 20011 x 2304 -> 768 104 us padded,
// 63 without), but for two cases: where an XCD's whole token tiles make one round of workgroups more
// than a range would (18000 x 192 -> 4608 1.09, 86400 x 8192 -> 768 1.14), and with weights of 5504
// rows or more and up to 4096 channels (86400 x 512 -> 11008 1.13, 172800 x 1536 -> 8192 1.05,
// 172800 x 2048 -> 6144 1.03, 172800 x 2752 -> 5504 1.03, below that 0.96-1.03; 86400 x 5504 -> 8192
// 0.93).
bool interleave_tiles(long long m_tiles, long long n_tiles, int K, int F) {
  if (F >= 5504 && K <= 4096) return false;
  auto rounds = [](long long tiles_of_an_xcd) { return (tiles_of_an_xcd + 31) / 32; };
  return rounds((m_tiles + 7) / 8 * n_tiles) == rounds((m_tiles * n_tiles + 7) / 8);
}
inline unsigned gemm_grid(const GemmParams& p) {
  const unsigned m = (unsigned)p.m_tiles;
  return (p.interleave ? (m + 7) / 8 * 8 : m) * (unsigned)p.n_tiles;
}

__device__ __forceinline__ float silu(float u) {
  return u * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-u * kLog2e));
}

// Where a workgroup's tile lies.
struct GemmTileAt {
  int sample, nt;
  int valid_rows;        // rows of the tile that exist
  long long row0;        // its first row
};
template <class Sh>
__device__ __forceinline__ bool gemm_tile_at(const GemmParams& p, int item, GemmTileAt& t) {
  int mt;
  if (!gemm_tile(p, item, mt, t.nt)) return false;
  t.sample = mt / p.m_tiles_per_sample;
  const int tile_in_sample = mt - t.sample * p.m_tiles_per_sample;
  t.row0 = (long long)t.sample * p.rows_per_sample + (long long)tile_in_sample * Sh::kBM;
  const long long rows_left = p.rows_per_sample - (long long)tile_in_sample * Sh::kBM;
  t.valid_rows = rows_left < Sh::kBM ? (int)rows_left : Sh::kBM;
  return true;
}

// Feature (weight row) of tile row R.  SwiGLU tiles pair kBN / 2 u-features with their
// v-features: wave column wn holds u rows in its first 32 tile rows, v rows in the next 32.
template <class Sh, bool kSwiglu>
__device__ __forceinline__ int gemm_feature(const GemmParams& p, int nt, int R) {
  if constexpr (kSwiglu) {
    const int hidden = p.F >> 1;
    int j = nt * (Sh::kBN / 2) + (R >> 6) * 32 + (R & 31);
    j = j < hidden ? j : hidden - 1;
    return ((R >> 5) & 1) ? hidden + j : j;
  }
  const int f = nt * Sh::kBN + R;
  return f < p.F ? f : p.F - 1;
}

// Row scale, bias, (gate); results pass through the LDS so that they leave in 16-byte pieces, eight
// lanes per 128-byte row segment.  Each wave stages its part, kStoreBlocks * 32 rows x 64 features at a
// time, in a region of its own at `stage_w` (128-byte rows, 16-byte chunks XORed with the row so that
// neither side meets a bank conflict).
template <class Sh, bool kSwiglu>
__device__ __forceinline__ void gemm_store(const GemmParams& p, const GemmTileAt& t, f32x16 (&acc)[2][Sh::NB],
                                           uint32_t stage_w, int wm, int wn, int lane) {
  constexpr int NB = Sh::NB, kBN = Sh::kBN, SB = Sh::kStoreBlocks;
  settle(lane);   // addresses are worked out here, not kept through the caller's loop over tiles
  const int li = lane & 31, g = lane >> 5;
  const int hidden = p.F >> 1;
  const float* bias = p.bias ? p.bias + (long long)t.sample * p.F : nullptr;
  auto position = [](int row, int chunk) __attribute__((always_inline)) {
    return (uint32_t)(row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
  };

  // writes the wave's staged block (`chunks` 16-byte chunks per row), whose first row is block b0's, to
  // `dst` (row pitch ld): chunk c of a row goes to column col_of(c)
  auto flush = [&](bf16_t* dst, long long ld, int chunks, int b0, auto col_of, int limit)
      __attribute__((always_inline)) {
    const int rows_per_inst = 64 / chunks;
    const int r_in = lane / chunks, c = lane % chunks;
    const int col = col_of(c);
#pragma unroll 4
    for (int i = 0; i < SB * 32 / rows_per_inst; ++i) {
      const int ml = i * rows_per_inst + r_in;
      const int m = wm * (NB * 32) + b0 * 32 + ml;
      const u32x4 v = *reinterpret_cast<const AERIS_LDS u32x4*>(stage_w + position(ml, c));
      if (m < t.valid_rows && col < limit)
        *reinterpret_cast<u32x4*>(dst + (t.row0 + m) * ld + col) = v;
    }
  };

  float rs[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    int m = wm * (NB * 32) + b * 32 + li;
    m = m < t.valid_rows ? m : t.valid_rows - 1;
    rs[b] = p.r ? p.r[t.row0 + m] : 1.f;
  }
  // four features from column `col` (a multiple of 4) of the lane's row in staged block b
  auto stage_store = [&](int b, int col, float o0, float o1, float o2, float o3)
      __attribute__((always_inline)) {
    u32x2 v = {pack_bf16(o0, o1), pack_bf16(o2, o3)};
    *reinterpret_cast<AERIS_LDS u32x2*>(stage_w + position(b * 32 + li, col >> 3) + (col & 4) * 2) = v;
  };

  if constexpr (kSwiglu) {
    const int jw = t.nt * (kBN / 2) + wn * 32;         // first gate column of this wave
    // u and v in place of the products; the fences here and below keep the compiler from working
    // on all of a wave's values at once, which spills
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      int j = jw + 8 * vq + 4 * g;
      j = j < hidden ? j : hidden - 4;
      const f32x4 bu = bias ? *reinterpret_cast<const f32x4*>(bias + j) : f32x4{0.f, 0.f, 0.f, 0.f};
      const f32x4 bv = bias ? *reinterpret_cast<const f32x4*>(bias + hidden + j) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[0][b][4 * vq + e] = __builtin_fmaf(acc[0][b][4 * vq + e], rs[b], bu[e]);
          acc[1][b][4 * vq + e] = __builtin_fmaf(acc[1][b][4 * vq + e], rs[b], bv[e]);
        }
      sched_fence();
    }
    if (p.y) {   // the optional uv output, staged as [u 32 | v 32]
#pragma unroll
      for (int b0 = 0; b0 < NB; b0 += SB) {
#pragma unroll
        for (int b = 0; b < SB; ++b)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const f32x16 &u = acc[0][b0 + b], &v = acc[1][b0 + b];
            stage_store(b, 8 * vq + 4 * g, u[4 * vq], u[4 * vq + 1], u[4 * vq + 2], u[4 * vq + 3]);
            stage_store(b, 32 + 8 * vq + 4 * g, v[4 * vq], v[4 * vq + 1], v[4 * vq + 2], v[4 * vq + 3]);
          }
        // chunk c: c < 4 -> u columns jw + 8c, else v columns hidden + jw + 8(c - 4); a column
        // past `hidden` (ragged last tile) is marked by F, which the limit rejects
        flush(p.y, p.F, 8, b0, [&](int c) {
          const int j = jw + 8 * (c & 3);
          return j < hidden ? (c < 4 ? j : hidden + j) : p.F;
        }, p.F);
      }
    }
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += SB) {
#pragma unroll
      for (int b = 0; b < SB; ++b)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          float o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = silu(acc[0][b0 + b][4 * vq + e]) * acc[1][b0 + b][4 * vq + e];
          stage_store(b, 8 * vq + 4 * g, o[0], o[1], o[2], o[3]);
          sched_fence();
        }
      flush(p.g, hidden, 4, b0, [&](int c) { return jw + 8 * c; }, hidden);
    }
  } else {
    const int fw = t.nt * kBN + wn * 64;               // first feature of this wave
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += SB) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          int f = fw + a * 32 + 8 * vq + 4 * g;
          f = f < p.F ? f : p.F - 4;
          const f32x4 b4 = bias ? *reinterpret_cast<const f32x4*>(bias + f) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int b = 0; b < SB; ++b) {
            const f32x16& v = acc[a][b0 + b];
            stage_store(b, a * 32 + 8 * vq + 4 * g, __builtin_fmaf(v[4 * vq], rs[b0 + b], b4[0]),
                        __builtin_fmaf(v[4 * vq + 1], rs[b0 + b], b4[1]),
                        __builtin_fmaf(v[4 * vq + 2], rs[b0 + b], b4[2]),
                        __builtin_fmaf(v[4 * vq + 3], rs[b0 + b], b4[3]));
          }
        }
      flush(p.y, p.F, 8, b0, [&](int c) { return fw + 8 * c; }, p.F);
    }
  }
}

template <class Sh>
__device__ __forceinline__ void gemm_clear(f32x16 (&acc)[2][Sh::NB]) {
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < Sh::NB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
}

// The two smaller shapes: one workgroup per tile, two per CU.  Bound by the latency of a step (copies,
// one barrier, the first operand reads), which the CU's other workgroup covers in part.  The loop is
// written out once per stage, so that every LDS offset is an immediate, with the order of products,
// reads and copies fenced: the compiler's own order was 4 to 7 % slower (9522 x 2944 -> 704 42.8 us, now
// 40.9; 4000 x 1024 -> 1024 11.9 / 11.5; 64 x 64 tiles 914 x 1600 -> 512 11.3 / 8.2).
template <class Sh, bool kSwiglu>
__global__ __launch_bounds__(Sh::kWaves * 64, 2) void norm_linear_gemm_kernel(GemmParams p) {
  constexpr int kBN = Sh::kBN, NB = Sh::NB, W = Sh::kWaves, kStages = Sh::kStages;
  constexpr int kPartBytes = Sh::kPartBytes, kStageBytes = Sh::kStageBytes;
  extern __shared__ __align__(16) unsigned char smem[];
  GemmTileAt at;
  if (!gemm_tile_at<Sh>(p, blockIdx.x, at)) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / Sh::WN, wn = wave % Sh::WN;
  const int li = lane & 31, g = lane >> 5;

  // ---- copies: instruction j moves rows 8j..8j+7 of the stage; wave w issues
  // j = w + W i.  i < 4: weight rows, i >= 4: token rows.  Rows past the end repeat the last
  // valid row (never stored).  Lane: row j*8 + lane/8, LDS chunk position lane%8.
  const bf16_t* wmat = p.w + (long long)at.sample * p.w_sample_stride;
  const unsigned long long wbase = reinterpret_cast<unsigned long long>(wmat);
  const unsigned long long xbase = reinterpret_cast<unsigned long long>(p.x + at.row0 * p.K);
  uint32_t voff[8];
  {
    const int r_in = lane >> 3;
    const int r_sub = ((wave & 1) << 3) | r_in;                  // row within a 64-row sub-tile, mod 16
    const int chunk = (lane & 7) ^ Sub::swz(r_sub);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int R = ((wave + W * i) << 3) + r_in;
      if (i < 4) {
        voff[i] = (uint32_t)((long long)gemm_feature<Sh, kSwiglu>(p, at.nt, R) * p.K * 2 + chunk * 16);
      } else {
        int m = R - kBN;
        m = m < at.valid_rows ? m : at.valid_rows - 1;
        voff[i] = (uint32_t)((long long)m * p.K * 2 + chunk * 16);
      }
    }
  }
  const uint32_t lds0 = lds_address(smem);
  auto copy_piece = [&](int i, uint32_t stage, int k0, uint32_t enable) __attribute__((always_inline)) {
    async_copy16_off(voff[i], (i < 4 ? wbase : xbase) + (unsigned long long)k0 * 2,
                     stage + (uint32_t)((wave + W * i) << 10), enable);
  };

  // ---- operand reads: per lane four chunk offsets (one per 16-channel block of a step)
  uint32_t va[4], vb[4];
  {
    const int s = Sub::swz(li);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint32_t off = li * 128 + (((2 * kk + g) ^ s) << 4);
      va[kk] = lds0 + wn * 8192 + off;
      vb[kk] = lds0 + kPartBytes + wm * (NB * 4096) + off;
    }
  }

  f32x16 acc[2][NB];
  gemm_clear<Sh>(acc);

  const int k_steps = p.K / kBK;
  // stages 0 .. kStages-2 are on their way before the first step
#pragma unroll
  for (int st = 0; st < kStages - 1; ++st)
#pragma unroll
    for (int i = 0; i < 8; ++i) copy_piece(i, lds0 + st * kStageBytes, st * kBK, st < k_steps);

  bf16x8 ao[2][2], bo[2][NB];
  auto fetch_a = [&](int set, int kk, uint32_t from) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 2; ++a) ao[set][a] = Sub::read_rm(va[kk] + from + a * 4096);
  };
  auto fetch_b = [&](int set, int kk, uint32_t from) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < NB; ++b) bo[set][b] = Sub::read_rm(vb[kk] + from + b * 4096);
  };
  // One step of 64 channels, in stage `slot`.
  auto step = [&](auto slot, int ks) __attribute__((always_inline)) {
    constexpr int kSlot = decltype(slot)::value;
    constexpr uint32_t kHere = kSlot * kStageBytes, kNext = (kSlot + kStages - 1) % kStages * kStageBytes;
    // This wave's copies of this stage have landed; those of up to kStages - 2 later stages
    // (eight each, in order) may still be on their way.
    if constexpr (kStages == 2) {
      wait_async_loads();
    } else {
      static_assert(kStages <= 4);
      const int later = k_steps - 1 - ks;
      if (kStages >= 4 && later >= 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
      else if (later >= 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      else wait_async_loads();
    }
    __syncthreads();               // this stage has landed; every reader of the stage before is done
    const uint32_t more = ks + kStages - 1 < k_steps;
    fetch_a(0, 0, kHere);
    fetch_b(0, 0, kHere);
    sched_fence();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int q = 0; q < 2 * NB; ++q) {
        const int a = q / NB, b = q % NB;
        acc[a][b] = mfma32(ao[kk & 1][a], bo[kk & 1][b], acc[a][b]);
        if (kk < 3 && q == 0) fetch_a((kk + 1) & 1, kk + 1, kHere);
        if (kk < 3 && q == (NB == 1 ? 0 : 1)) fetch_b((kk + 1) & 1, kk + 1, kHere);
        // the copies of a later stage, the one that the last step's readers have left, ride in the first
        // half of the step, spread over its products, so that they have the second half to land before
        // the wait that opens the next step
        if (kk < 2) {
          const int n = kk * 2 * NB + q;
#pragma unroll
          for (int i = n * 2 / NB; i < (n + 1) * 2 / NB; ++i)
            copy_piece(i, lds0 + kNext, (ks + kStages - 1) * kBK, more);
        }
        sched_fence();
      }
    }
  };
  static_assert(kStages == 2 || kStages == 4);
  for (int ks = 0;;) {
    step(Const<0>{}, ks);
    if (++ks == k_steps) break;
    step(Const<1>{}, ks);
    if (++ks == k_steps) break;
    if constexpr (kStages == 4) {
      step(Const<2>{}, ks);
      if (++ks == k_steps) break;
      step(Const<3>{}, ks);
      if (++ks == k_steps) break;
    }
  }

  __syncthreads();                                   // every wave is done with the operand stages
  gemm_store<Sh, kSwiglu>(p, at, acc, lds0 + wave * Sh::kStoreBytes, wm, wn, lane);
}

// The 256 x 256 shape: one workgroup of eight wavefronts per CU, which walks over its tiles.
//
// Bound by the board's power cap (MFMA pipes busy 79 % of the cycles at 1.62 GHz).  A loop in which all
// eight waves fetch and multiply together left the pipes idle at every barrier and first fetch (65 % busy
// at 1.80 GHz).  Here the two waves of a SIMD take turns: a step is two halves of 16 products, and waves
// 4-7 run one barrier behind waves 0-3, so that one multiplies while the other fetches its operands and
// issues copies.  A half of a stage is copied over as soon as both waves have its operands in registers,
// up to seven halves (3000 cycles) ahead of its use, so the waits count copies and hardly ever wait.
// The last steps of a tile fetch the first of the next one, and its results, staged in the operand stage
// just left, are stored while the next tile is multiplied: a tile costs 5.7 us beside its steps where
// separate workgroups took 9.  Per call, us, all waves together / in turns of 8 products,
// a workgroup per tile / as here, one session: 172800 x 2048 -> 6144 3644 / 3480 / 3292;
// 172800 x 5504 -> 2048 3229 / 2965 / 2796; 32400 x 1024 -> 3072 185 / 184 / 171.  With
// v_mfma_f32_16x16x32_bf16, which alone runs cooler, it takes 1.05 times as long.
template <bool kSwiglu>
__global__ __launch_bounds__(GemmLarge::kWaves * 64, 2) void projection_gemm_kernel(GemmParams p) {
  using Sh = GemmLarge;
  constexpr uint32_t kStageBytes = Sh::kStageBytes, kHalfBytes = kStageBytes / 4;
  extern __shared__ __align__(16) unsigned char smem[];
  GemmTileAt at;
  int item = blockIdx.x;
  if (!gemm_tile_at<Sh>(p, item, at)) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / Sh::WN, wn = wave % Sh::WN;
  const int li = lane & 31, g = lane >> 5;
  const uint32_t lds0 = lds_address(smem);

  // ---- copies.  A stage is four halves of 128 rows: weight rows 0, 1, token rows 2, 3; half h holds
  // the h-th 32 of every 64 features (the u or the v features of a SwiGLU tile) and the h-th 64 of
  // every 128 token rows, so that a wave's part of the tile is 64 features x 128 rows side by side.
  // Wave w issues instructions w and w + 8 of a half, 8 rows each; lane: row lane / 8, LDS chunk
  // position lane % 8.  Rows past the end repeat the last valid row (never stored).
  unsigned long long wbase, xbase;
  uint32_t voff[8];
  auto sources = [&](const GemmTileAt& t) __attribute__((always_inline)) {
    int lane_ = lane;
    settle(lane_);
    wbase = reinterpret_cast<unsigned long long>(p.w + (long long)t.sample * p.w_sample_stride);
    xbase = reinterpret_cast<unsigned long long>(p.x + t.row0 * p.K);
    const int chunk = (lane_ & 7) ^ Sub::swz(((wave & 1) << 3) | (lane_ >> 3));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = i >> 1, r = ((wave + 8 * (i & 1)) << 3) + (lane_ >> 3);   // row of the half
      const int f = gemm_feature<Sh, kSwiglu>(p, t.nt, (r >> 5) * 64 + h * 32 + (r & 31));
      int m = (r >> 6) * 128 + h * 64 + (r & 63);
      m = m < t.valid_rows ? m : t.valid_rows - 1;
      voff[i] = (uint32_t)f * (uint32_t)(p.K * 2) + chunk * 16;
      voff[4 + i] = (uint32_t)m * (uint32_t)(p.K * 2) + chunk * 16;
    }
  };
  auto copy_half = [&](int half, uint32_t stage, int step) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      async_copy16_at(voff[2 * half + i], (half < 2 ? wbase : xbase) + (unsigned long long)step * (kBK * 2),
                      lds0 + stage + half * kHalfBytes + ((wave + 8 * i) << 10));
  };

  // ---- operand reads: per lane four chunk offsets (one per 16-channel block of a step)
  uint32_t va[4], vb[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const uint32_t off = li * 128 + (((2 * kk + g) ^ Sub::swz(li)) << 4);
    va[kk] = lds0 + wn * 4096 + off;
    vb[kk] = lds0 + 2 * kHalfBytes + wm * 8192 + off;
  }

  f32x16 acc[2][4];
  bf16x8 w0[4], w1[4], x[2][4];
  auto fetch_w = [&](bf16x8 (&w)[4], uint32_t from) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) w[kk] = Sub::read_rm(va[kk] + from);
  };
  auto fetch_x = [&](uint32_t from) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int b = 0; b < 2; ++b) x[b][kk] = Sub::read_rm(vb[kk] + from + b * 4096);
  };
  // all but the newest `behind` copies of this wave have landed
  auto landed = [&](auto behind) __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(behind)::value) : "memory");
  };
  auto meet = [&]() __attribute__((always_inline)) {
    sched_fence();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    sched_fence();
  };
  // Token rows of half h by all 64 features: 16 products between two meetings, while the other wave of the
  // SIMD fetches.  Reads are complete when a wave meets the others, so that copies issued after a meeting
  // may overwrite what was read before it.
  auto products = [&](int h) __attribute__((always_inline)) {
    meet();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        acc[0][2 * h + b] = mfma32(w0[kk], x[b][kk], acc[0][2 * h + b]);
        acc[1][2 * h + b] = mfma32(w1[kk], x[b][kk], acc[1][2 * h + b]);
      }
    __builtin_amdgcn_s_setprio(0);
    meet();
  };

  const int k_steps = p.K / kBK;
  GemmTileAt next;
  bool follows = false, first_tile = true;        // follows: another tile after this one
  sources(at);
  copy_half(0, 0, 0);
  copy_half(1, 0, 0);
  copy_half(2, 0, 0);
  copy_half(3, 0, 0);
  if (k_steps > 1) {
    copy_half(0, kStageBytes, 1);
    copy_half(1, kStageBytes, 1);
    copy_half(2, kStageBytes, 1);
    landed(Const<8>{});
  } else {
    landed(Const<2>{});
  }
  meet();
  if (wm == 1) meet();
  gemm_clear<Sh>(acc);
  uint32_t here = 0;
  for (int t = 0;;) {
    const bool fresh = t == 0 && !first_tile;     // the whole step has landed
    if (t == 0) follows = k_steps > 1 && gemm_tile_at<Sh>(p, item + gridDim.x, next);
    if (!fresh)
      for (; t + 2 < k_steps; ++t, here = kStageBytes - here) {
        fetch_w(w0, here);
        fetch_w(w1, here + kHalfBytes);
        fetch_x(here);
        copy_half(3, kStageBytes - here, t + 1);
        landed(Const<8>{});
        products(0);
        fetch_x(here + kHalfBytes);
        copy_half(0, here, t + 2);
        copy_half(1, here, t + 2);
        copy_half(2, here, t + 2);
        landed(Const<8>{});
        products(1);
      }
    const uint32_t other = kStageBytes - here;
    const int left = k_steps - 1 - t;             // steps of this tile after this one
    fetch_w(w0, here);
    fetch_w(w1, here + kHalfBytes);
    fetch_x(here);
    if (left >= 1 || follows) {
      copy_half(3, other, left >= 1 ? t + 1 : 0);
      if (!fresh) landed(Const<8>{});
    } else {
      landed(Const<0>{});
    }
    products(0);
    fetch_x(here + kHalfBytes);
    if (left >= 2 || (left == 1 && follows)) {
      if (left == 1) sources(next);
      const int ahead = left >= 2 ? t + 2 : 0;
      copy_half(0, here, ahead);
      copy_half(1, here, ahead);
      copy_half(2, here, ahead);
      landed(Const<8>{});
    } else if (left == 1) {
      landed(Const<2>{});
    } else {
      landed(Const<0>{});
    }
    products(1);

    if (left == 0) {
      if (wm == 0) meet();
      gemm_store<Sh, kSwiglu>(p, at, acc, lds0 + here + wave * Sh::kStoreBytes, wm, wn, lane);
      if (!follows) return;
      meet();          // every wave has read its results back: the stage may be filled again
      gemm_clear<Sh>(acc);
      copy_half(0, here, 1);
      copy_half(1, here, 1);
      copy_half(2, here, 1);
      if (wm == 1) meet();
      at = next;
      item += gridDim.x;
      first_tile = false;
      t = 0;
    } else {
      ++t;
    }
    here = other;
  }
}

// r_i = (mean_c x_ic^2 + eps)^(-1/2): one wavefront per row, 16 bytes per lane and access.  Workgroup
// `block` of `blocks`.
__device__ __forceinline__ void rms_rows(const bf16_t* __restrict__ x, long long n_rows, int channels, float eps,
                                         float* __restrict__ r, unsigned block, unsigned blocks) {
  const int lane = threadIdx.x & 63;
  const long long wave = (long long)block * 4 + (threadIdx.x >> 6);
  const long long n_waves = (long long)blocks * 4;
  for (long long row = wave; row < n_rows; row += n_waves) {
    const bf16_t* xr = x + row * channels;
    float s = 0.f;
    for (int c = lane * 8; c < channels; c += 512) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c);
#pragma unroll
      for (int e = 0; e < 8; ++e) s = __builtin_fmaf((float)v[e], (float)v[e], s);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    if (lane == 0) r[row] = 1.f / sqrtf(s / (float)channels + eps);
  }
}

// Wf_b[f][c] = bf16(W[f][c] w[c] (1 + gamma_b[c])),  bias_b[f] = sum_c beta_b[c] W[f][c].
// One workgroup per (feature, sample); the bias sum is taken in a fixed order.
__device__ __forceinline__ void fold_weights(const bf16_t* __restrict__ w_in, const float* __restrict__ w,
                                             const float* __restrict__ gamma, const float* __restrict__ beta,
                                             int K, int F, bf16_t* __restrict__ w_out,
                                             float* __restrict__ bias, int f, long long b) {
  __shared__ float part[4];
  const bf16_t* src = w_in + (long long)f * K;
  bf16_t* dst = w_out + (b * F + f) * K;
  float s = 0.f;
  for (int c = threadIdx.x * 8; c < K; c += 256 * 8) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(src + c);
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float wv = (float)v[e];
      o[e] = (bf16_t)(wv * (w[c + e] * (1.f + gamma[b * K + c + e])));
      s = __builtin_fmaf(beta[b * K + c + e], wv, s);
    }
    *reinterpret_cast<bf16x8*>(dst + c) = o;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) bias[b * F + f] = (part[0] + part[1]) + (part[2] + part[3]);
}

// Both in one launch, which leaves one to wait for instead of two and runs them side by side (each is
// bound by latency: a few rows per wave, one row of weights per workgroup).  In x a share of the row blocks
// first, then a block per feature; samples in y.  One launch of 40 fewer per projection in a small
// layer, whose host side is the bound (see between_kernel in linear_bwd.hip); two samples of 16,200 rows x
// 1024, 3072 and 5504 features, four projections: 742 -> 737 us.
__global__ __launch_bounds__(256) void norm_fold_kernel(
    const bf16_t* __restrict__ x, long long n_rows, float eps, float* __restrict__ r, unsigned row_blocks,
    const bf16_t* __restrict__ w_in, const float* __restrict__ w, const float* __restrict__ gamma,
    const float* __restrict__ beta, int K, int F, bf16_t* __restrict__ w_out, float* __restrict__ bias) {
  if (blockIdx.x >= row_blocks) fold_weights(w_in, w, gamma, beta, K, F, w_out, bias, (int)(blockIdx.x - row_blocks), blockIdx.y);
  else rms_rows(x, n_rows, K, eps, r, blockIdx.y * row_blocks + blockIdx.x, gridDim.y * row_blocks);
}

size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }

}  // namespace

int projection_gemm_check(long long n_rows, long long rows_per_sample, int K, int F) {
  if (n_rows <= 0 || rows_per_sample <= 0 || K < kBK || F < 8) return AERIS_ERR_INVALID_SHAPE;
  if (K % kBK != 0 || F % 8 != 0 || n_rows % rows_per_sample != 0) return AERIS_ERR_NOT_DIVISIBLE;
  if (n_rows / rows_per_sample > 65535) return AERIS_ERR_INVALID_SHAPE;   // a grid dimension
  // 32-bit byte offsets inside a workgroup's operand tiles, 31-bit tile counts
  if ((long long)F * K * 2 >= (1LL << 32)) return AERIS_ERR_INVALID_SHAPE;
  const long long m_tiles = (n_rows / rows_per_sample) *
                            ((rows_per_sample + GemmLarge::kBM - 1) / GemmLarge::kBM);
  const long long n_tiles = (F + GemmLarge::kBN - 1) / GemmLarge::kBN;
  if (((m_tiles + 63) / 64) * 64 * n_tiles >= (1LL << 31)) return AERIS_ERR_INVALID_SHAPE;
  return AERIS_OK;
}

namespace {

int check_projection(int64_t n_rows, int64_t rows_per_sample, int32_t channels, int32_t features) {
  if (n_rows <= 0 || rows_per_sample <= 0 || channels <= 0 || features <= 0)
    return AERIS_ERR_INVALID_SHAPE;
  if (channels > AERIS_MAX_PROJECTION_CHANNELS) return AERIS_ERR_INVALID_SHAPE;
  return projection_gemm_check(n_rows, rows_per_sample, channels, features);
}

bool bad16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) != 0; }

}  // namespace

namespace {

// Fills in the tile counts of a shape; false if its grid does not fit a launch.
template <class Sh>
bool gemm_tiles(GemmParams& p) {
  const long long per_sample = (p.rows_per_sample + Sh::kBM - 1) / Sh::kBM;
  const long long m_tiles = per_sample * p.n_samples;
  const int features = p.swiglu ? p.F / 2 : p.F, tile = p.swiglu ? Sh::kBN / 2 : Sh::kBN;
  p.n_tiles = (features + tile - 1) / tile;
  if ((m_tiles + 63) / 64 * 64 * p.n_tiles >= (1LL << 31)) return false;
  p.m_tiles_per_sample = (int)per_sample;
  p.m_tiles = (int)m_tiles;
  p.interleave = Sh::NB == 4 && interleave_tiles(m_tiles, p.n_tiles, p.K, p.F);
  return true;
}

template <class Sh, bool kSwiglu>
int launch_gemm_kernel(const GemmParams& p, hipStream_t stream) {
  if constexpr (std::is_same<Sh, GemmLarge>::value) {
    // one workgroup per CU, which walks its tiles (every 256th); all of them where a tile has too few
    // steps to look into the next one
    const unsigned items = gemm_grid(p);
    if (!allow_full_lds<projection_gemm_kernel<kSwiglu>>()) return -1;
    return launch_kernel(projection_gemm_kernel<kSwiglu>, dim3(p.K > kBK && items > kCus ? kCus : items),
                         dim3(Sh::kWaves * 64), (size_t)Sh::kSmem, stream, p);
  } else {
    if (!allow_full_lds<norm_linear_gemm_kernel<Sh, kSwiglu>>()) return -1;
    return launch_kernel(norm_linear_gemm_kernel<Sh, kSwiglu>, dim3(gemm_grid(p)),
                         dim3(Sh::kWaves * 64), (size_t)Sh::kSmem, stream, p);
  }
}
template <class Sh>
int launch_gemm_shape(const GemmParams& p, hipStream_t stream) {
  return p.swiglu ? launch_gemm_kernel<Sh, true>(p, stream) : launch_gemm_kernel<Sh, false>(p, stream);
}

// Which tile shape: the one whose rounds of workgroups are estimated to end first, from the time a
// round takes (microseconds: a fixed part plus a part per 64-channel step, less of both for a last
// round that leaves CUs empty).  Medium tiles fetch the rows twice as often as large ones, which
// counts once rows and results exceed the last-level cache (300000 x 192 -> 576 145 us with large
// tiles, 161 with medium ones; 60000 x 192 -> 1408 67 / 58).  With 64 channels a large tile is a single step that
// overlaps nothing: medium tiles were the faster ones at all sizes of more than one round of large tiles (large /
// medium 9165 x 64 -> 2944 21.2 / 19.1, 105886 x 64 -> 192 19.4 / 18.0, 26387 x 64 -> 6144 82.7 / 77.0, 699334 x 64 ->
// 896 352 / 286), and by up to 5 % below.  Fitted to 200 sizes of 1500 ... 150000 rows, 64 ... 5760 channels and 128
// ... 6400 features; at 417 others (700 ... 200000 rows, 64 ... 2048 channels, 64 ... 6400 features, operands in the
// last-level cache and out of it) what it takes is 1 % slower than the best shape on average, more than 5 % at 22
// of them.  Small tiles have the shortest steps and are taken as long
// as each has a CU of its own: 914 rows x 1600 -> 512 takes 8.2 us with small, 12.7 with medium tiles, 1759 x
// 640 -> 1344 (588 small tiles) 11.0 and 7.8.  Medium tiles win while large ones leave more than about half
// of the CUs without work (9522 x 2944 -> 704, 114 large tiles: 41 / 57), large ones, with half the operand
// bytes per product, from there on (148, 18926 x 2560 -> 512: 70 / 53; 150, 12738 x 5248 -> 704: 133 / 99;
// 172800 x 2048 -> 2048: 1391 / 1097).
enum class GemmTile { kLarge, kMedium, kSmall };
constexpr long long kNoTiles = 1LL << 40;   // of a count that does not fit a launch: rules the finer tiles out
GemmTile choose_gemm_tile(long long large_tiles, long long medium_tiles, long long small_tiles, int steps,
                          bool cached) {
  if (small_tiles <= (long long)kCus) return GemmTile::kSmall;
  if (steps == 1 && large_tiles > (long long)kCus && medium_tiles < kNoTiles) return GemmTile::kMedium;
  // one large workgroup per CU, two medium ones
  const double large_rest = (double)(large_tiles % kCus) / kCus;
  const double large = (double)(large_tiles / kCus) * (5.7 + 1.45 * steps) +
                       (large_rest > 0.0 ? 7.2 + steps * (0.83 + 0.85 * large_rest * large_rest) : 0.0);
  const double medium_rest = (double)(medium_tiles % (2 * kCus)) / (2 * kCus);
  const double medium = (double)(medium_tiles / (2 * kCus)) * (2.5 + 0.93 * steps) +
                        (medium_rest > 0.0 ? 4.8 + steps * (0.42 + 0.45 * medium_rest) : 0.0);
  return medium * (cached ? 1.0 : 1.2) < large ? GemmTile::kMedium : GemmTile::kLarge;
}

}  // namespace

namespace {

// Fills in p's tile counts for the shape that is taken, false if no shape fits a launch.
bool plan_gemm(GemmParams& p, GemmTile& tile) {
  GemmParams large = p, medium = p, small = p;
  if (!gemm_tiles<GemmLarge>(large)) return false;
  auto tiles = [](bool fits, const GemmParams& q) { return fits ? (long long)q.m_tiles * q.n_tiles : kNoTiles; };
  const bool cached = (double)p.n_samples * p.rows_per_sample * ((double)p.K + p.F) * 2.0 <= 256e6;
  tile = choose_gemm_tile(tiles(true, large), tiles(gemm_tiles<GemmMedium>(medium), medium),
                          tiles(gemm_tiles<GemmSmall>(small), small), p.K / kBK, cached);
  p = tile == GemmTile::kLarge ? large : tile == GemmTile::kMedium ? medium : small;
  return true;
}

}  // namespace

int launch_projection_gemm(GemmParams p, hipStream_t stream) {
  GemmTile tile;
  if (!plan_gemm(p, tile)) return -1;
  switch (tile) {
    case GemmTile::kSmall: return launch_gemm_shape<GemmSmall>(p, stream);
    case GemmTile::kMedium: return launch_gemm_shape<GemmMedium>(p, stream);
    default: return launch_gemm_shape<GemmLarge>(p, stream);
  }
}

namespace {

struct Folded {
  bf16_t* w;
  float* bias;
  float* r;
};
Folded carve(void* workspace, int64_t n_rows, int64_t n_samples, int32_t channels, int32_t features) {
  char* ws = static_cast<char*>(workspace);
  Folded f;
  f.w = reinterpret_cast<bf16_t*>(ws);
  ws += round256((size_t)n_samples * features * channels * 2);
  f.bias = reinterpret_cast<float*>(ws);
  ws += round256((size_t)n_samples * features * 4);
  f.r = reinterpret_cast<float*>(ws);
  return f;
}

// Row pass + weight folding + GEMM.  features = rows of `weight`; swiglu: features = 2 * hidden.
int norm_projection(const void* x, const float* w, const float* gamma, const float* beta, float eps,
                    const void* weight, int64_t n_rows, int64_t rows_per_sample, int32_t channels,
                    int32_t features, bool swiglu, void* y, void* g, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
  if (!x || !w || !gamma || !beta || !weight || !workspace || (!swiglu && !y) || (swiglu && !g))
    return AERIS_ERR_NULL_POINTER;
  if (const int rc = check_projection(n_rows, rows_per_sample, channels, features)) return rc;
  if (!(eps >= 0.f)) return AERIS_ERR_INVALID_SHAPE;
  if (bad16(x) || bad16(weight) || bad16(y) || bad16(g) || bad16(workspace) || bad16(w) ||
      bad16(gamma) || bad16(beta))
    return AERIS_ERR_MISALIGNED;
  if (workspace_bytes < aeris_norm_linear_workspace_bytes(n_rows, rows_per_sample, channels, features))
    return AERIS_ERR_WORKSPACE_TOO_SMALL;
  const hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int64_t n_samples = n_rows / rows_per_sample;
  const Folded f = carve(workspace, n_rows, n_samples, channels, features);
  const long long waves = (n_rows + 3) / 4;
  unsigned row_blocks = (unsigned)(((waves < 8192 ? waves : 8192) + n_samples - 1) / n_samples);
  // a launch holds less than 2^32 work items along x: nearly that many features leave room for few row blocks
  constexpr unsigned kMostBlocks = 0xffffffffu / 256;
  if ((unsigned)features < kMostBlocks && row_blocks > kMostBlocks - (unsigned)features)
    row_blocks = kMostBlocks - (unsigned)features;
  if (launch_kernel(norm_fold_kernel, dim3(row_blocks + (unsigned)features, (unsigned)n_samples), dim3(256), 0,
                    st, static_cast<const bf16_t*>(x), (long long)n_rows, eps, f.r, row_blocks,
                    static_cast<const bf16_t*>(weight), w, gamma, beta, channels, features, f.w, f.bias) != 0)
    return AERIS_ERR_HIP_LAUNCH;
  GemmParams p{};
  p.x = static_cast<const bf16_t*>(x);
  p.w = f.w;
  p.w_sample_stride = (long long)features * channels;
  p.r = f.r;
  p.bias = f.bias;
  p.y = static_cast<bf16_t*>(y);
  p.g = static_cast<bf16_t*>(g);
  p.rows_per_sample = rows_per_sample;
  p.n_samples = n_samples;
  p.K = channels;
  p.F = features;
  p.swiglu = swiglu ? 1 : 0;
  return launch_projection_gemm(p, st) == 0 ? AERIS_OK : AERIS_ERR_HIP_LAUNCH;
}

}  // namespace
}  // namespace aeris

using namespace aeris;

extern "C" size_t aeris_norm_linear_workspace_bytes(int64_t n_rows, int64_t rows_per_sample,
                                                    int32_t channels, int32_t out_features) {
  if (check_projection(n_rows, rows_per_sample, channels, out_features) != AERIS_OK) return 0;
  const size_t n_samples = (size_t)(n_rows / rows_per_sample);
  return round256(n_samples * out_features * channels * 2) + round256(n_samples * out_features * 4) +
         round256((size_t)n_rows * 4);
}

extern "C" int aeris_norm_linear_fwd(const void* x, const float* w, const float* gamma,
                                     const float* beta, float eps, const void* weight,
                                     int64_t n_rows, int64_t rows_per_sample, int32_t channels,
                                     int32_t out_features, void* y, void* workspace,
                                     size_t workspace_bytes, void* hip_stream) {
  return norm_projection(x, w, gamma, beta, eps, weight, n_rows, rows_per_sample, channels,
                         out_features, false, y, nullptr, workspace, workspace_bytes, hip_stream);
}

extern "C" int aeris_norm_linear_swiglu_fwd(const void* x, const float* w, const float* gamma,
                                            const float* beta, float eps, const void* weight,
                                            int64_t n_rows, int64_t rows_per_sample,
                                            int32_t channels, int32_t hidden, void* g, void* uv,
                                            void* workspace, size_t workspace_bytes,
                                            void* hip_stream) {
  if (hidden <= 0 || hidden > (1 << 29)) return AERIS_ERR_INVALID_SHAPE;
  if (hidden % 8 != 0) return AERIS_ERR_NOT_DIVISIBLE;
  return norm_projection(x, w, gamma, beta, eps, weight, n_rows, rows_per_sample, channels,
                         2 * hidden, true, uv, g, workspace, workspace_bytes, hip_stream);
}

extern "C" int aeris_linear_fwd(const void* x, const void* weight, int64_t n_rows, int32_t channels,
                                int32_t out_features, void* y, void* hip_stream) {
  if (!x || !weight || !y) return AERIS_ERR_NULL_POINTER;
  if (const int rc = check_projection(n_rows, n_rows, channels, out_features)) return rc;
  if (bad16(x) || bad16(weight) || bad16(y)) return AERIS_ERR_MISALIGNED;
  GemmParams p{};
  p.x = static_cast<const bf16_t*>(x);
  p.w = static_cast<const bf16_t*>(weight);
  p.y = static_cast<bf16_t*>(y);
  p.rows_per_sample = n_rows;
  p.n_samples = 1;
  p.K = channels;
  p.F = out_features;
  return launch_projection_gemm(p, static_cast<hipStream_t>(hip_stream)) == 0 ? AERIS_OK : AERIS_ERR_HIP_LAUNCH;
}

extern "C" int aeris_projection_plan(int64_t n_rows, int64_t rows_per_sample, int32_t channels,
                                     int32_t features, int32_t gated, int32_t* tile, int32_t* in_turn) {
  if (!tile || !in_turn) return AERIS_ERR_NULL_POINTER;
  if (const int rc = check_projection(n_rows, rows_per_sample, channels, features)) return rc;
  if (gated && features % 16 != 0) return AERIS_ERR_NOT_DIVISIBLE;
  GemmParams p{};
  p.rows_per_sample = rows_per_sample;
  p.n_samples = n_rows / rows_per_sample;
  p.K = channels;
  p.F = features;
  p.swiglu = gated ? 1 : 0;
  GemmTile t;
  if (!plan_gemm(p, t)) return AERIS_ERR_INVALID_SHAPE;
  *tile = t == GemmTile::kLarge ? 256 : t == GemmTile::kMedium ? 128 : 64;
  *in_turn = p.interleave;
  return AERIS_OK;
}
