// Backward attention of short windows in one kernel: one workgroup owns a whole (batch, window, head)
// and makes dQ, dK and dV of it (same contract as launch_bwd, statistics in the workspace included).  dQ
// alone, and dK and dV alone, are builds of the same kernel without the other's work: stages give the bits of
// the whole.  (A selection at run time in one build cost the whole 1 to 7 %.)  dQ with its statistics and then dK
// and dV, us, the two kernels of longer windows / these two: 8 heads of 32, 16 tokens 218 / 124, 64: 81 / 82,
// 120: 90 / 124, 144: 135 / 131, 192: 107 / 145; 7 of 64, 64 tokens 167 / 163, 120: 162 / 196, 144: 242 / 214.
//
// Short windows are bound by memory and its latency, and the two kernels of longer windows serve them
// badly: 14 passes over tensors and seven products where 8 and five would do, tiles of 128 resident tokens
// of which 16 or 144 - 128 exist, and a load that nothing overlaps in front of a few blocks of work.  Here
// Q, dO and K of the window go to the LDS at once (V and O to registers) and stay there.  Per block of
// 32 queries each wave computes S, dP, P and dS of its keys and adds to its dV and dK, which need no
// exchange; dS passes through a strip [keys][32 queries] in the LDS, from which the waves make dQ of the
// block, in pieces of 16 queries x 32 channels.  Keys are dealt to the waves in units of 16
// (v_mfma_f32_16x16x32_bf16): in blocks of 32 a window of 144 would need five waves, and a workgroup of
// five is given room as one of eight (one workgroup per CU instead of two, 254 us instead of 176).
// The barrier of a block waits for the LDS alone, and the loads of the prologue are unconditional: each
// kept the stores of dQ, or one load at a time, in flight instead of all (loads: 207 -> 185 us).
//
// Backward call, us, two kernels / this one (8 heads of 32, 7 of 64, 3 of 128; 65,000 tokens):
//   tokens          8          16         25         49         64        100        144        176
//   head_dim 32  418 / 101  218 /  84  149 /  84   99 /  70   83 / 64    94 /  87  135 /  92  116 / 107
//   head_dim 64  822 / 152  454 / 114  314 / 107  193 / 117  164 / 106  177 / 149  256 / 164
//   head_dim 128 569 / 168  318 / 118  230 / 103  163 / 116  145 / 103
// 12 x 12 windows, 8 heads of 64 on 180 x 360: 300 -> 176 us, 530 MB in and out, 3.0 TB/s.  Left: the
// loop's own latency (barrier, LDS round trips, 24,000 of 42,000 cycles of a workgroup) with two
// workgroups per CU to hide it.
#include "winattn_common.hpp"
#include "winattn_launch.hpp"

namespace aeris {

// Rows of the LDS arrays: whole blocks of 32 queries.
__host__ __device__ inline int short_rows(int T) { return (T + 31) & ~31; }
// Units of 16 keys.
__host__ __device__ inline int short_units(int T) { return (T + 15) >> 4; }

// Q, dO, K | two strips of dS, [keys][32 queries] | LSE * log2(e), delta | token table.  Strips are read in
// whole blocks of 32 keys: where keys end in the middle of one, a read of the second strip runs on into what
// lies behind it (and is cleared in the register), which for 33 to 48 tokens is shorter than that.
constexpr size_t short_smem_bytes(int T, int D) {
  const size_t rows = (T + 31) & ~31, keys = (T + 15) & ~15;
  const size_t arrays = 2 * keys * 64 + 3 * rows * 4, read = (keys + rows) * 64;
  return 3 * rows * D * 2 + (arrays > read ? arrays : read);
}
// The last byte that a block of the second strip reads, as the kernel forms its addresses.
constexpr bool short_strip_reads_fit(int D) {
  for (int T = 1; T <= 192; ++T) {
    const size_t rows = (T + 31) & ~31, units = (T + 15) >> 4, n_blocks = rows >> 5;
    const size_t second = 3 * rows * D * 2 + units * 16 * 64;
    if (second + (n_blocks - 1) * (32 * 64) + 32 * 64 > short_smem_bytes(T, D)) return false;
  }
  return true;
}
static_assert(short_strip_reads_fit(32) && short_strip_reads_fit(64) && short_strip_reads_fit(128));

// Waves a SIMD must hold (beside what the LDS allows).
template <int D, int NU>
constexpr int kShortWaves = D == 32 ? (NU == 1 ? 4 : 3) : D == 64 ? (NU == 1 ? 3 : 2) : 2;

template <int kCtrl>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}

// NU: units of 16 keys per wave, W wavefronts.  kStages: 7, or 2 (dQ), or 4 (dK, dV), which take the statistics
// from the workspace unless told to make them.
template <int D, int NU, typename OutT, int kStages>
__global__ __launch_bounds__(256, (kShortWaves<D, NU>)) void winattn_bwd_short_kernel(
    KParams p, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ d_o, const OutT* __restrict__ o, const float* __restrict__ lse,
    float* __restrict__ delta, float* __restrict__ lse2v, OutT* __restrict__ dq, OutT* __restrict__ dk,
    OutT* __restrict__ dv, int make) {
  constexpr bool kDq = kStages & 2, kDkDv = kStages & 4;
  const bool make_stats = kStages == 7 || make != 0;
  using Tl = Tile<D>;
  using Strip = Tile<32>;
  constexpr int kKK = D / 32, kCB = D / 16;               // products over channels; blocks of 16 channels
  constexpr uint32_t kBlockBytes = 32 * D * 2, kHalfBytes = 16 * D * 2;   // 32, 16 token rows
  constexpr int kRowsPerInst = Tl::kRowsPerInst;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, W = blockDim.x >> 6;
  const int lane = tid & 63, hw_wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // The first waves have a unit more than the last where units do not divide: of the workgroups that share
  // a CU they sit on different SIMDs.
  const int wave = W == 4 ? (hw_wave + 2 * ((blockIdx.x >> 8) & 1)) & 3 : hw_wave;
  const int li = lane & 15, g = lane >> 4;

  int pair, tile;
  if (!block_to_work(p, pair, tile)) return;
  if (make_stats && blockIdx.x == 0)   // padding behind the last pair, as the other kernels leave it
    for (int t = tid; t < kStream; t += blockDim.x) {
      delta[(long long)p.n_pairs * p.T + t] = 0.f;
      lse2v[(long long)p.n_pairs * p.T + t] = 0.f;
    }
  Window win;
  if (!win.init(p, pair)) {
    for (int t = tid; make_stats && t < p.T; t += blockDim.x) {   // a skipped window still gets finite statistics
      delta[(long long)pair * p.T + t] = 0.f;
      lse2v[(long long)pair * p.T + t] = 0.f;
    }
    return;
  }
  const int rows = short_rows(p.T), units = short_units(p.T);
  const uint32_t array_bytes = rows * D * 2, strip_bytes = units * 16 * 64;
  const uint32_t lds0 = lds_address(smem);
  const uint32_t q_at = lds0, do_at = q_at + array_bytes, k_at = do_at + array_bytes;
  const uint32_t strips = k_at + array_bytes, stat_at = strips + 2 * strip_bytes;
  const uint32_t table = stat_at + 2 * rows * 4;

  const long long plane = (long long)p.H * p.W;
  const long long qkv_base = ((long long)win.b * plane) * p.qkv_tok + (long long)win.head * p.qkv_head;
  const long long q_base = ((long long)win.b * plane) * p.q_tok + (long long)win.head * p.q_head;
  const long long k_base = ((long long)win.b * plane) * p.k_tok + (long long)win.head * p.k_head;
  const long long o_base = ((long long)win.b * plane) * p.o_tok + (long long)win.head * p.o_head;

  for (int t = tid; t < rows; t += blockDim.x)
    *reinterpret_cast<AERIS_LDS int*>(table + t * 4) = win.grid_index(p, t < p.T ? t : p.T - 1);
  lds_barrier();
  auto grid_of = [&](int t) __attribute__((always_inline)) {
    return (unsigned)*reinterpret_cast<const AERIS_LDS int*>(table + t * 4);
  };

  // ---- everything is on its way at once: Q, dO and K to the LDS, this wave's keys of V and this
  // thread's share of O to registers
  {
    const char* qs = reinterpret_cast<const char*>(q + q_base);
    const char* dos = reinterpret_cast<const char*>(d_o + o_base);
    const char* ks = reinterpret_cast<const char*>(k + k_base);
    const uint32_t q_row = (uint32_t)(p.q_tok * 2), o_row = (uint32_t)(p.o_tok * 2), k_row = (uint32_t)(p.k_tok * 2);
    // 1 KB, kRowsPerInst rows, at a time; the waves in turn
    // rows / W is 32 at most with one wave, 64 NU / 4 with four
    constexpr int kMost = (NU < 2 ? 32 : 16 * NU) / kRowsPerInst;
    const int n_inst = rows / kRowsPerInst;
    unsigned at[kMost];
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
      const int n = wave + W * i;
      at[i] = grid_of((n < n_inst ? n : 0) * kRowsPerInst + lane / Tl::NC);
    }
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
      const int n = wave + W * i;
      if (n >= n_inst) break;
      const int chunk = ((lane % Tl::NC) ^ Tl::swz(n * kRowsPerInst + lane / Tl::NC)) * 16;
      async_copy16(ks + (unsigned long long)at[i] * k_row + chunk, k_at + n * 1024);
      async_copy16(dos + (unsigned long long)at[i] * o_row + chunk, do_at + n * 1024);
      async_copy16(qs + (unsigned long long)at[i] * q_row + chunk, q_at + n * 1024);
    }
  }
  struct Unit {
    int w_lo, w_hi, lo_max, hi_min;       // queries that see any, and all, of its keys
  } unit[NU];
  bf16x8 vreg[NU][kKK], kreg[NU][kKK];
#pragma unroll
  for (int i = 0; i < NU; ++i) {
    const int first = (wave + W * i) * 16, own = first + li, last = first + 15;
    int lo, hi;
    Unit& un = unit[i];
    un.w_lo = un.w_hi = un.lo_max = un.hi_min = 0;
    if (first < p.T) {
      win.range(first, lo, hi);
      un.w_lo = lo;
      un.hi_min = hi;
      win.range(last < p.T ? last : p.T - 1, lo, hi);
      un.w_hi = hi;
      un.lo_max = last < p.T ? lo : 1 << 30;             // phantom keys: never free of the mask
    }
    const bf16_t* row = v + qkv_base + (long long)grid_of(own < p.T ? own : p.T - 1) * p.qkv_tok + 8 * g;
#pragma unroll
    for (int kk = 0; kk < kKK; ++kk) vreg[i][kk] = *reinterpret_cast<const bf16x8*>(row + 32 * kk);
    un.w_lo = __builtin_amdgcn_readfirstlane(un.w_lo);
    un.w_hi = __builtin_amdgcn_readfirstlane(un.w_hi);
    un.lo_max = __builtin_amdgcn_readfirstlane(un.lo_max);
    un.hi_min = __builtin_amdgcn_readfirstlane(un.hi_min);
  }
  const uint32_t rm = q_at + Tl::chunk_offset(li, g);     // row-major: row lane % 16, chunk lane / 16
  {
    // delta = sum_c dO O, D / 8 threads per token, with the summation tree of winattn_delta_kernel
    constexpr int kChunks = D / 8, kPasses = NU * kChunks / 4;
    const int c = tid % kChunks, per_pass = blockDim.x / kChunks;
    Raw8<OutT> o8[kPasses];
#pragma unroll
    for (int i = 0; i < kPasses && make_stats; ++i) {
      const int t = i * per_pass + tid / kChunks;
      const long long at = grid_of(t < p.T ? t : p.T - 1);
      o8[i].load(o + o_base + at * p.o_tok + 8 * c);
    }
    const float own_lse =
        make_stats ? lse[((long long)win.b * p.nh + win.head) * plane + grid_of(tid < p.T ? tid : p.T - 1)] : 0.f;
    for (int t = p.T + tid; t < rows; t += blockDim.x) {   // phantom queries: finite statistics
      *reinterpret_cast<AERIS_LDS float*>(stat_at + t * 4) = 0.f;
      *reinterpret_cast<AERIS_LDS float*>(stat_at + (rows + t) * 4) = 0.f;
    }
    wait_async_loads();
    __syncthreads();
    if (!make_stats && tid < p.T)
      *reinterpret_cast<AERIS_LDS float*>(stat_at + (rows + tid) * 4) = delta[(long long)pair * p.T + tid];
    if (tid < p.T) {
      const float l2 = make_stats ? own_lse * kLog2e : lse2v[(long long)pair * p.T + tid];
      *reinterpret_cast<AERIS_LDS float*>(stat_at + tid * 4) = l2;
      if (make_stats) lse2v[(long long)pair * p.T + tid] = l2;
    }
#pragma unroll
    for (int i = 0; i < kPasses && make_stats; ++i) {
      const int t = i * per_pass + tid / kChunks;
      if (t < p.T) {   // whole token groups leave together
        const bf16x8 d8 = Tl::read_rm(do_at + Tl::chunk_offset(t, c));
        float a[8], acc = 0.f;
        o8[i].values(a);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = __builtin_fmaf(a[e], (float)d8[e], acc);
        acc += dpp<0xB1>(acc);                             // lane ^ 1
        acc += dpp<0x4E>(acc);                             // lane ^ 2
        if (kChunks > 4) acc += dpp<0x141>(acc);           // lane ^ 7 (the sums of a quad are equal)
        if (kChunks > 8) acc += dpp<0x140>(acc);           // lane ^ 15
        if (c == 0) {
          *reinterpret_cast<AERIS_LDS float*>(stat_at + (rows + t) * 4) = acc;
          delta[(long long)pair * p.T + t] = acc;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NU; ++i)
#pragma unroll
      for (int kk = 0; kk < kKK; ++kk) {
        const int u = wave + W * i;
        kreg[i][kk] = Tl::read_rm((rm ^ (uint32_t)(kk << 6)) + 2 * array_bytes + (u < units ? u : 0) * kHalfBytes);
      }
    lds_barrier();
  }

  f32x4 dkacc[NU][kCB], dvacc[NU][kCB];
#pragma unroll
  for (int i = 0; i < NU; ++i)
#pragma unroll
    for (int c = 0; c < kCB; ++c) dkacc[i][c] = dvacc[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  // transposing reads of Q and dO (queries 4g.. and 16 + 4g.. of a block, the order that the logits of a
  // lane have), and of K and the strip (keys 8g..): a 16-lane block fetches four rows at a time
  const int l4r = li >> 2, l4c = (li & 3) >> 1, l4h = (li & 1) * 8;
  const uint32_t tr = q_at + Tl::chunk_offset(4 * g + l4r, l4c) + l4h;
  const uint32_t tk = k_at + Tl::chunk_offset(8 * g + l4r, l4c) + l4h;
  const uint32_t ts = strips + Strip::chunk_offset(8 * g + l4r, l4c) + l4h;
  // where a lane puts its key's dS: queries 4g.. and 16 + 4g.. of the key's row
  const uint32_t ds_at = strips + Strip::chunk_offset(li, g >> 1) + (g & 1) * 8;

  const int n_blocks = rows >> 5;
  int turn = wave;
  for (int j = 0; j < n_blocks; ++j) {
    const uint32_t strip_off = (j & 1) * strip_bytes, off = j * kBlockBytes;
    bf16x8 qa[2][kKK], doa[2][kKK];
    f32x4 l2[2], dl[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int kk = 0; kk < kKK; ++kk) {
        const uint32_t at = (rm ^ (uint32_t)(kk << 6)) + off + h * kHalfBytes;
        qa[h][kk] = Tl::read_rm(at);
        doa[h][kk] = Tl::read_rm(at + array_bytes);
      }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t at = stat_at + (j * 32 + 16 * h + 4 * g) * 4;
      l2[h] = *reinterpret_cast<const AERIS_LDS f32x4*>(at);
      dl[h] = *reinterpret_cast<const AERIS_LDS f32x4*>(at + rows * 4);
    }
    union Packed { u32x4 u; bf16x8 h; };
    Packed pb[NU], dsb[NU];
    unsigned seen = 0;                                    // bit i: queries of the block see unit i
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      const Unit& un = unit[i];
      const int s0 = j * 32;
      if (s0 + 32 <= un.w_lo || s0 >= un.w_hi) {
        pb[i].u = dsb[i].u = u32x4{0, 0, 0, 0};
        continue;
      }
      seen |= 1u << i;
      f32x4 s[2], dp[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) s[h] = dp[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < kKK; ++kk)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          s[h] = mfma16(qa[h][kk], kreg[i][kk], s[h]);
          dp[h] = mfma16(doa[h][kk], vreg[i][kk], dp[h]);
        }
      if (!(s0 >= un.lo_max && s0 + 32 <= un.hi_min)) {
        asm volatile("");                                  // a branch, not a select for every element
        const int own = (wave + W * i) * 16 + li;
        int lo, hi;
        win.range(own, lo, hi);
        if (own >= p.T) hi = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int qidx = s0 + 16 * h + 4 * g + e;
            if (qidx < lo || qidx >= hi) s[h][e] = -INFINITY;
          }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float pr[4], ds[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          pr[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h][e], p.scale_log2, -l2[h][e]));
          ds[e] = pr[e] * (dp[h][e] - dl[h][e]);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          pb[i].u[2 * h + e] = pack_bf16(pr[2 * e], pr[2 * e + 1]);
          dsb[i].u[2 * h + e] = pack_bf16(ds[2 * e], ds[2 * e + 1]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      const int u = wave + W * i;
      if (kDq && u < units) {
        const uint32_t at = ds_at + u * (16 * 64) + strip_off;
        *reinterpret_cast<AERIS_LDS u32x2*>(at) = u32x2{dsb[i].u[0], dsb[i].u[1]};
        *reinterpret_cast<AERIS_LDS u32x2*>(at ^ 32) = u32x2{dsb[i].u[2], dsb[i].u[3]};
      }
    }
    // Queries that none of a unit's keys sees are left out: zero times an infinity is no zero.  All operands
    // are read in front of the branches (a second loop for blocks that only some units see spilled; operands
    // cleared by masks: head_dim 64, 81 tokens 144.4 -> 151.0 us).
    seen = __builtin_amdgcn_readfirstlane(seen);
    bf16x8 dot[kCB], qt[kCB];
#pragma unroll
    for (int c = 0; c < kCB; ++c) {
      const uint32_t at = (tr ^ (uint32_t)(c << 5)) + off;
      dot[c] = Tl::read_tr(at + array_bytes, at + array_bytes + kHalfBytes);
      qt[c] = Tl::read_tr(at, at + kHalfBytes);
    }
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      if (!kDkDv || !(seen >> i & 1)) continue;
#pragma unroll
      for (int c = 0; c < kCB; ++c) {
        dvacc[i][c] = mfma16(dot[c], pb[i].h, dvacc[i][c]);
        dkacc[i][c] = mfma16(qt[c], dsb[i].h, dkacc[i][c]);
      }
    }
    if constexpr (!kDq) continue;
    // the strip is complete; the one of the block before is free again
    lds_barrier();
    // ---- dQ of these 32 queries: pieces of 16 queries x 32 channels, dealt to the waves in turn
    for (int u = turn; u < kCB; u += W) {
      const int half = u & 1, cb = u >> 1;
      const uint32_t k0 = tk ^ (uint32_t)(cb << 6), s0 = (ts ^ (uint32_t)(half << 5)) + strip_off;
      f32x4 acc[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      // Operands of several products on their way at a time: a chain of LDS latencies otherwise.
      constexpr int kBatch = NU >= 3 ? 3 : 2 * NU;
      // the blocks of 32 keys that any of the queries sees; the others are left out like queries above
      int n_begin = 0, n_end = n_blocks;
      if (n_blocks > 1) {
        int lo, hi, unused;
        const int first = j * 32 + half * 16, last = first + 15 < p.T ? first + 15 : p.T - 1;
        win.range(first, lo, unused);
        win.range(last, unused, hi);
        n_begin = lo >> 5;
        n_end = (hi + 31) >> 5;
      }
#pragma unroll 1
      for (int n0 = n_begin; n0 < n_end; n0 += kBatch) {
        bf16x8 ka[kBatch][2], sb[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          const int m = n0 + i < n_end ? n0 + i : n_end - 1;
          const uint32_t kn = k0 + m * kBlockBytes, sn = s0 + m * (32 * 64);
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const uint32_t at = kn ^ (uint32_t)(c << 5);
            ka[i][c] = Tl::read_tr(at, (at ^ 16) + 4 * D * 2);
          }
          sb[i] = Strip::read_tr(sn, (sn ^ 16) + 4 * 64);
        }
        sched_fence();
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          if (n0 + i >= n_end) break;
          // a last block of which the strip holds only 16 keys
          if (n0 + i == n_blocks - 1 && (units & 1)) {
            asm volatile("");
            if (g >= 2) sb[i] = bf16x8{};
          }
#pragma unroll
          for (int c = 0; c < 2; ++c) acc[c] = mfma16(ka[i][c], sb[i], acc[c]);
        }
      }
      const int t = j * 32 + half * 16 + li;
      if (t < p.T) {
        const int at = grid_of(t);
        OutT* row = dq + qkv_base + (long long)at * p.qkv_tok;
        float p_lat = 0.f, p_lon = 0.f;
        if (p.rope) rope_position(p, at, p_lat, p_lon);
        float e[2][4];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
          for (int i = 0; i < 4; ++i) e[c][i] = acc[c][i] * p.scale;
          if (p.rope)
            rope_unrotate4(e[c][0], e[c][1], e[c][2], e[c][3], cb * 32 + c * 16 + 4 * g, p_lat, p_lon, p.rope_c);
        }
        store_blocks(row + cb * 32, g, e[0], e[1]);
      }
    }
    turn -= kCB % W;
    if (turn < 0) turn += W;
  }
  if constexpr (!kDkDv) return;

#pragma unroll
  for (int i = 0; i < NU; ++i) {
    const int own = (wave + W * i) * 16 + li;
    if (own >= p.T) continue;
    const int at = grid_of(own);
    OutT* dkrow = dk + qkv_base + (long long)at * p.qkv_tok;
    OutT* dvrow = dv + qkv_base + (long long)at * p.qkv_tok;
    float p_lat = 0.f, p_lon = 0.f;
    if (p.rope) rope_position(p, at, p_lat, p_lon);
#pragma unroll
    for (int c = 0; c < kCB; c += 2) {
      float e[2][4], f[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          e[h][n] = dkacc[i][c + h][n] * p.scale;
          f[h][n] = dvacc[i][c + h][n];
        }
        if (p.rope)
          rope_unrotate4(e[h][0], e[h][1], e[h][2], e[h][3], (c + h) * 16 + 4 * g, p_lat, p_lon, p.rope_c);
      }
      store_blocks(dkrow + 16 * c, g, e[0], e[1]);
      store_blocks(dvrow + 16 * c, g, f[0], f[1]);
    }
  }
}

// Waves of a workgroup, and units of keys per wave.
inline int short_waves(int T) { return short_units(T) < 4 ? short_units(T) : 4; }
inline int short_units_per_wave(int T) { return (short_units(T) + short_waves(T) - 1) / short_waves(T); }

template <int D, int NU, typename OutT>
static int launch_short_t(KParams kp, const void* q, const void* k, const void* v, const void* o, const float* lse,
                          const void* d_o, float* delta, float* lse2, void* dq, void* dk, void* dv,
                          hipStream_t stream, unsigned stages) {
  kp.n_tiles = 1;
  kp.n_whole = whole_short_windows(kp, AttnKernel::kDkDv, D);
  auto launch = [&](auto which, int make) {
    constexpr int kStages = decltype(which)::value;
    if (!allow_full_lds<winattn_bwd_short_kernel<D, NU, OutT, kStages>>()) return -1;
    return launch_kernel(winattn_bwd_short_kernel<D, NU, OutT, kStages>, dim3(grid_blocks(kp)),
                         dim3(short_waves(kp.T) * 64), short_smem_bytes(kp.T, D), stream, kp,
                         static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k), static_cast<const bf16_t*>(v),
                         static_cast<const bf16_t*>(d_o), static_cast<const OutT*>(o), lse, delta, lse2,
                         static_cast<OutT*>(dq), static_cast<OutT*>(dk), static_cast<OutT*>(dv), make);
  };
  if (stages == 7u) return launch(Const<7>{}, 1);
  const int make = stages & 1u;
  if (!(stages & 4u)) return launch(Const<2>{}, make);
  if (!(stages & 2u)) return launch(Const<4>{}, make);
  return launch(Const<2>{}, make) == 0 ? launch(Const<4>{}, 0) : -1;
}

// Windows that leave room for a second workgroup in a CU's LDS, with at most three units of keys per wave:
// up to 192 tokens at head_dim 32, 144 at 64, 64 at 128.  A workgroup alone has nothing to overlap its loads
// with: two kernels / this one, head_dim 64 169 tokens 225 / 232 us, head_dim 128 81 tokens 164 / 271, 128
// tokens 148 / 212; four units per wave (head_dim 32, 196 tokens: 132 / 189) spill.
bool short_backward(const KParams& kp, int head_dim) {
  return short_units(kp.T) <= 12 && 2 * short_smem_bytes(kp.T, head_dim) <= 160 * 1024;
}

int launch_bwd_short(const KParams& kp, int head_dim, bool out_f32, const void* q, const void* k, const void* v,
                     const void* o, const float* lse, const void* d_o, float* delta, float* lse2, void* dq,
                     void* dk, void* dv, hipStream_t stream, unsigned stages) {
#define AERIS_SHORT_CASE(DD, NN)                                                                              \
  if (head_dim == DD && short_units_per_wave(kp.T) == NN)                                                     \
    return out_f32                                                                                                \
               ? launch_short_t<DD, NN, float>(kp, q, k, v, o, lse, d_o, delta, lse2, dq, dk, dv, stream, stages) \
               : launch_short_t<DD, NN, bf16_t>(kp, q, k, v, o, lse, d_o, delta, lse2, dq, dk, dv, stream, stages);
  AERIS_SHORT_CASE(32, 1)
  AERIS_SHORT_CASE(32, 2)
  AERIS_SHORT_CASE(32, 3)
  AERIS_SHORT_CASE(64, 1)
  AERIS_SHORT_CASE(64, 2)
  AERIS_SHORT_CASE(64, 3)
  AERIS_SHORT_CASE(128, 1)
#undef AERIS_SHORT_CASE
  return -1;
}

}  // namespace aeris
