// Forward attention of short windows: a workgroup holds the keys and values of a whole (batch, window,
// head); its queries are its own, or where there are few windows and heads dealt to two or three workgroups
// (same contract as launch_fwd).
//
// Bound by memory and its latency.  K and V go to the LDS at once, queries to registers, and nothing is
// streamed: a wave computes the logits of 16 queries with every key (v_mfma_f32_16x16x32_bf16, a lane has
// all keys of one query but for an exchange among four lanes), takes the maximum and the exponentials once,
// and multiplies with V.  No barrier after the loads, no rescaling, and units of 16 queries instead of
// tiles of 128 of which 16 or 144 - 128 exist.
//
// us, streamed tiles / this kernel (8 heads of 32, 7 of 64, 3 of 128; 65,000 tokens):
//   tokens           16         25         36         49         64         81        144        176
//   head_dim 32    99 / 35    67 / 35    53 / 36    41 / 30    33 / 25    39 / 29   57 / 36    46 / 39
//   head_dim 64   117 / 38    79 / 37    62 / 39    50 / 37    44 / 37    51 / 44   69 / 57    58 / 54
//   head_dim 128  115 / 33    80 / 32    62 / 36    52 / 33    47 / 32    52 / 41
#include "winattn_common.hpp"
#include "winattn_launch.hpp"

namespace aeris {

// K, V | token table
constexpr size_t fwd_short_smem_bytes(int blocks, int D) { return 2 * (size_t)blocks * 32 * D * 2 + (size_t)blocks * 32 * 4; }

__device__ __forceinline__ float row_pair_max(float x) {   // over lanes l, l ^ 16
  const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// NB: blocks of 32 keys.  kShared: p.n_tiles workgroups share a window and head (a build of its own: with the
// division of work in scalar registers the other is up to 6 % slower, 81 tokens, head_dim 64, 4096 windows and
// heads 32.2 -> 33.8 us, 96 tokens 34.2 -> 36.4).
template <int D, int NB, typename OutT, bool kShared>
__global__ __launch_bounds__(256, 2) void winattn_fwd_short_kernel(
    KParams p, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    OutT* __restrict__ o, float* __restrict__ lse) {
  using Tl = Tile<D>;
  constexpr int kKK = D / 32, kCB = D / 16;               // products over channels; blocks of 16 channels
  constexpr int kUnits = (2 * NB + 3) / 4;                // units of 16 queries per wave, at most
  constexpr uint32_t kHalfBytes = 16 * D * 2, kArrayBytes = NB * 32 * D * 2;
  constexpr int kRowsPerInst = Tl::kRowsPerInst, kInst = NB * 32 / kRowsPerInst;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, W = blockDim.x >> 6;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, g = lane >> 4;

  int pair, tile;
  if (!block_to_work(p, pair, tile)) return;
  // units of 16 queries are dealt to the waves of all workgroups of the pair in turn
  const int unit0 = kShared ? tile * W + wave : wave, unit_step = kShared ? p.n_tiles * W : W;
  Window win;
  if (!win.init(p, pair)) return;
  const uint32_t k_at = lds_address(smem), v_at = k_at + kArrayBytes, table = v_at + kArrayBytes;
  for (int t = tid; t < NB * 32; t += blockDim.x)
    *reinterpret_cast<AERIS_LDS int*>(table + t * 4) = win.grid_index(p, t < p.T ? t : p.T - 1);
  lds_barrier();
  auto grid_of = [&](int t) __attribute__((always_inline)) {
    return (unsigned)*reinterpret_cast<const AERIS_LDS int*>(table + t * 4);
  };

  const long long plane = (long long)p.H * p.W;
  const long long q_base = ((long long)win.b * plane) * p.q_tok + (long long)win.head * p.q_head;
  const long long k_base = ((long long)win.b * plane) * p.k_tok + (long long)win.head * p.k_head;
  const long long v_base = ((long long)win.b * plane) * p.qkv_tok + (long long)win.head * p.qkv_head;
  {
    const char* ks = reinterpret_cast<const char*>(k + k_base);
    const char* vs = reinterpret_cast<const char*>(v + v_base);
    const uint32_t k_row = (uint32_t)(p.k_tok * 2), v_row = (uint32_t)(p.qkv_tok * 2);
    // 1 KB, kRowsPerInst rows, at a time; the waves in turn.  One wave has NB = 1 only, four any.
    constexpr int kMost = NB == 1 ? kInst : NB == 2 ? (kInst + 2) / 3 : (kInst + 3) / 4;
    unsigned at[kMost];
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
      const int n = wave + W * i;
      at[i] = grid_of((n < kInst ? n : 0) * kRowsPerInst + lane / Tl::NC);
    }
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
      const int n = wave + W * i;
      if (n >= kInst) break;
      const int chunk = ((lane % Tl::NC) ^ Tl::swz(n * kRowsPerInst + lane / Tl::NC)) * 16;
      async_copy16(ks + (unsigned long long)at[i] * k_row + chunk, k_at + n * 1024);
      async_copy16(vs + (unsigned long long)at[i] * v_row + chunk, v_at + n * 1024);
    }
  }
  bf16x8 qreg[kUnits][kKK];
  unsigned own[kUnits];
#pragma unroll
  for (int i = 0; i < kUnits; ++i) {
    const int t = (unit0 + unit_step * i) * 16 + li;
    own[i] = grid_of(t < p.T ? t : p.T - 1);
    const bf16_t* row = q + q_base + (long long)own[i] * p.q_tok + 8 * g;
#pragma unroll
    for (int kk = 0; kk < kKK; ++kk) qreg[i][kk] = *reinterpret_cast<const bf16x8*>(row + 32 * kk);
  }
  const uint32_t rm = k_at + Tl::chunk_offset(li, g);     // row-major: row lane % 16, chunk lane / 16
  // transposing reads of V: keys 4g.. and 16 + 4g.. of a block, the order that the logits of a lane have
  const uint32_t tr = v_at + Tl::chunk_offset(4 * g + (li >> 2), (li & 3) >> 1) + (li & 1) * 8;
  wait_async_loads();
  __syncthreads();

  // `count` units from the from-th of this wave, which share every operand read.  Two at a time where a
  // row is long (head_dim 128, 100 / 128 tokens: 46.9 / 41.7 us -> 43.6 / 39.3), one after the other where
  // that only makes the chain from logits to output longer (head_dim 32, 100 tokens 32.0 -> 36.2).
  constexpr bool kPairs = D == 128 && kUnits == 2;
  auto attend = [&](auto from, auto count) __attribute__((always_inline)) {
    constexpr int kFrom = decltype(from)::value, N = decltype(count)::value;
    // visible keys: of the lane, of all, and of any of its unit's queries
    int lo[N], hi[N], lo_max[N], hi_min[N], w_lo[N], w_hi[N];
    bool sees_all = true;                                 // every unit sees keys of every block
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = kFrom + u, first = (unit0 + unit_step * i) * 16, last = first + 15, t = first + li;
      if (p.rope) {   // rotary embedding of the queries
        float p_lat, p_lon;
        rope_position(p, own[i], p_lat, p_lon);
#pragma unroll
        for (int kk = 0; kk < kKK; ++kk)
          qreg[i][kk] = rope_rotate8(qreg[i][kk], kk * 32 + 8 * g, p_lat, p_lon, p.rope_c, false);
        if (p.q_rot_out && t < p.T) {   // by-product for the backward pass: no second rotation
          bf16_t* keep = p.q_rot_out + (((long long)win.b * plane + own[i]) * p.nh + win.head) * D + 8 * g;
#pragma unroll
          for (int kk = 0; kk < kKK; ++kk) *reinterpret_cast<bf16x8*>(keep + 32 * kk) = qreg[i][kk];
        }
      }
      win.range(first, w_lo[u], hi_min[u]);
      win.range(last < p.T ? last : p.T - 1, lo_max[u], w_hi[u]);
      win.range(t < p.T ? t : p.T - 1, lo[u], hi[u]);
      lo_max[u] = __builtin_amdgcn_readfirstlane(lo_max[u]);
      hi_min[u] = __builtin_amdgcn_readfirstlane(hi_min[u]);
      w_lo[u] = __builtin_amdgcn_readfirstlane(w_lo[u]);
      w_hi[u] = __builtin_amdgcn_readfirstlane(w_hi[u]);
      sees_all = sees_all && w_lo[u] < 32 && w_hi[u] > 32 * (NB - 1);
    }

    // logits, transposed: a lane has keys 4g.. of every 16, for one query of each unit
    f32x4 s[N][2 * NB];
#pragma unroll
    for (int n = 0; n < 2 * NB; ++n) {
      bf16x8 ka[kKK];
#pragma unroll
      for (int kk = 0; kk < kKK; ++kk) ka[kk] = Tl::read_rm((rm ^ (uint32_t)(kk << 6)) + n * kHalfBytes);
#pragma unroll
      for (int u = 0; u < N; ++u) {
        s[u][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < kKK; ++kk) s[u][n] = mfma16(ka[kk], qreg[kFrom + u][kk], s[u][n]);
        if (!(16 * n >= lo_max[u] && 16 * n + 16 <= hi_min[u])) {
          asm volatile("");                                // a branch, not a select for every element
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int kidx = 16 * n + 4 * g + e;
            if (kidx < lo[u] || kidx >= hi[u]) s[u][n][e] = -INFINITY;
          }
        }
      }
    }
    union Packed { u32x4 u; bf16x8 h; };
    Packed pb[N][NB];
    float mx[N], l[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      float m = s[u][0][0];
#pragma unroll
      for (int n = 0; n < 2 * NB; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) m = fmaxf(m, s[u][n][e]);
      mx[u] = wave_half_max(row_pair_max(m)) * p.scale_log2;
      const float m_sub = mx[u] == -INFINITY ? 0.f : mx[u];
      l[u] = 0.f;   // in fp32 over the unrounded probabilities
#pragma unroll
      for (int n = 0; n < 2 * NB; ++n) {
        float pv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          pv[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][n][e], p.scale_log2, -m_sub));
          l[u] += pv[e];
        }
        pb[u][n >> 1].u[2 * (n & 1)] = pack_bf16(pv[0], pv[1]);
        pb[u][n >> 1].u[2 * (n & 1) + 1] = pack_bf16(pv[2], pv[3]);
      }
      const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(l[u]), __float_as_uint(l[u]), false, false);
      l[u] = __uint_as_float(a[0]) + __uint_as_float(a[1]);
      const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(l[u]), __float_as_uint(l[u]), false, false);
      l[u] = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    }
    f32x4 acc[N][kCB];
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int c = 0; c < kCB; ++c) acc[u][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // V rows of blocks that no query of a unit sees are left out: zero times an infinity is no zero.  The first
    // operands are read in front of the branch, under the exponentials.  us, all rows multiplied / this / without
    // those first reads / branches alone, block by block, in every window: 7 heads of 64, 81 tokens 40.3 / 40.3 /
    // 40.8 / 42.5, 144: 50.7 / 51.2 / 51.5 / 50.8, 156: 49.6 / 51.1 / 51.9 / 50.6; 3 of 128, 81 tokens 36.0 / 36.2 /
    // 36.5 / 40.7; 16 of 32, 144 tokens 300.9 / 302.8 / 303.8 / 320.7.
    bf16x8 v0[kCB];
#pragma unroll
    for (int c = 0; c < kCB; ++c) v0[c] = Tl::read_tr(tr ^ (uint32_t)(c << 5), (tr ^ (uint32_t)(c << 5)) + kHalfBytes);
    auto outputs = [&](auto all) __attribute__((always_inline)) {
      constexpr bool kAll = decltype(all)::value != 0;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int u0 = 0; u0 < (kAll ? 1 : N); ++u0) {
          if (!kAll && (32 * b + 32 <= w_lo[u0] || 32 * b >= w_hi[u0])) continue;
#pragma unroll
          for (int c = 0; c < kCB; ++c) {
            const uint32_t at = (tr ^ (uint32_t)(c << 5)) + 2 * b * kHalfBytes;
            const bf16x8 va = b == 0 ? v0[c] : Tl::read_tr(at, at + kHalfBytes);
#pragma unroll
            for (int u = u0; u < (kAll ? N : u0 + 1); ++u) acc[u][c] = mfma16(va, pb[u][b].h, acc[u][c]);
          }
        }
    };
    if (NB == 1 || sees_all) outputs(Const<1>{});
    else outputs(Const<0>{});
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = kFrom + u;
      if ((unit0 + unit_step * i) * 16 + li < p.T) {
        const float inv = 1.f / l[u];
        OutT* row = o + ((long long)win.b * plane + own[i]) * p.o_tok + (long long)win.head * p.o_head;
#pragma unroll
        for (int c = 0; c < kCB; c += 2) {
          float a[2][4];
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[h][e] = acc[u][c + h][e] * inv;
          store_blocks(row + 16 * c, g, a[0], a[1]);
        }
        if (g == 0)
          lse[((long long)win.b * p.nh + win.head) * plane + own[i]] =
              (mx[u] + __builtin_amdgcn_logf(l[u])) * 0.6931471805599453f;
      }
    }
  };
  const int units = (p.T + 15) >> 4;
  if (kShared && unit0 >= units) return;
  if constexpr (kPairs) {
    if (unit0 + unit_step < units) attend(Const<0>{}, Const<2>{});
    else attend(Const<0>{}, Const<1>{});
  } else {
    attend(Const<0>{}, Const<1>{});
    if constexpr (kUnits >= 2) {
      if (unit0 + unit_step < units) attend(Const<1>{}, Const<1>{});
    }
    if constexpr (kUnits >= 3) {
      if (unit0 + 2 * unit_step < units) attend(Const<2>{}, Const<1>{});
    }
  }
}

// Workgroups that share the queries of a window and head: as many as leave each wave one unit of 16, while
// one for each would leave a part of the 256 CUs without work (from 161 tokens on, three units per wave, also
// at twice that).  Every workgroup loads all keys and values.  The waves do for a unit what they do alone.
// us, streamed tiles / one workgroup / as here, 2 heads:
//   windows x heads            32                   128                   256                   512
//   head_dim 32,  96 tokens   6.1 / 4.9 / 3.8      6.2 / 5.1 / 4.1      6.4 / 5.3 / 4.7      7.5 /  6.2
//                144          7.6 / 8.0 / 4.8      7.7 / 8.1 / 5.5      9.3 / 8.4 / 6.5     13.0 /  9.9
//                192          7.2 / 8.4 / 4.8      7.4 / 8.7 / 5.8      8.7 / 9.0 / 7.0     12.0 / 11.1 / 10.5
//   head_dim 64, 144          8.8 / 8.9 / 5.4      8.9 / 9.0 / 6.3     11.4 / 9.5 / 7.6     16.1 / 12.5
//                192          8.5 / 9.6 / 5.4      8.8 / 9.8 / 6.6     10.3 / 10.3 / 8.3    16.0 / 16.9 / 15.2
//   head_dim 128, 128         9.1 / 7.7 / 5.9      9.5 / 8.1 / 6.5     10.7 / 9.2 / 8.8     17.0 / 16.6
// At twice the limits: 96 tokens 512 6.2 -> 6.5, 144 tokens head_dim 64 512 12.5 -> 12.9, 192 tokens head_dim
// 32 1024 17.2 -> 17.2, 64 27.6 -> 26.2 but 176 tokens 768 13.9 -> 14.7.
int short_forward_workgroups(const KParams& kp) {
  const int units = (kp.T + 15) / 16;
  return kp.n_pairs <= (units > 10 ? 512 : 256) ? (units + 3) / 4 : 1;
}

template <int D, int NB, typename OutT>
static int launch_fwd_short_t(KParams kp, const void* q, const void* k, const void* v, void* o, float* lse,
                              hipStream_t stream) {
  kp.n_tiles = short_forward_workgroups(kp);
  kp.n_whole = whole_short_windows(kp, AttnKernel::kForward, D);
  const int units = (kp.T + 15) / 16;
  auto launch = [&](auto shared) {
    constexpr bool kShared = decltype(shared)::value != 0;
    if (!allow_full_lds<winattn_fwd_short_kernel<D, NB, OutT, kShared>>()) return -1;
    return launch_kernel(winattn_fwd_short_kernel<D, NB, OutT, kShared>, dim3(grid_blocks(kp)),
                         dim3((units < 4 ? units : 4) * 64), fwd_short_smem_bytes(NB, D), stream, kp,
                         static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k),
                         static_cast<const bf16_t*>(v), static_cast<OutT*>(o), lse);
  };
  if constexpr (NB >= 3) {
    if (kp.n_tiles > 1) return launch(Const<1>{});
  }
  return launch(Const<0>{});
}

// Windows of up to 192 tokens that leave room for a second workgroup in a CU's LDS (128 tokens at head_dim
// 128); above, 196 tokens at head_dim 32 take as long either way.  At head_dim 64 windows of 97 to 128
// tokens fill the streamed kernel's tile of 128 queries, which reads an operand for 32 queries where this
// reads it for 16: 121 tokens 45.4 / 48.6 us, 128 tokens 43.9 / 46.1.  By window and head_dim alone: a window
// has the same bits in every grid, batch and list of windows.
bool short_forward(const KParams& kp, int head_dim) {
  const int blocks = (kp.T + 31) / 32;
  if (head_dim == 64 && blocks == 4) return false;
  return blocks <= 6 && 2 * fwd_short_smem_bytes(blocks, head_dim) <= 160 * 1024;
}

int launch_fwd_short(const KParams& kp, int head_dim, bool out_f32, const void* q, const void* k, const void* v,
                     void* o, float* lse, hipStream_t stream) {
#define AERIS_SHORT_CASE(DD, NN)                                                          \
  if (head_dim == DD && (kp.T + 31) / 32 == NN)                                           \
    return out_f32 ? launch_fwd_short_t<DD, NN, float>(kp, q, k, v, o, lse, stream)       \
                   : launch_fwd_short_t<DD, NN, bf16_t>(kp, q, k, v, o, lse, stream);
  AERIS_SHORT_CASE(32, 1)
  AERIS_SHORT_CASE(32, 2)
  AERIS_SHORT_CASE(32, 3)
  AERIS_SHORT_CASE(32, 4)
  AERIS_SHORT_CASE(32, 5)
  AERIS_SHORT_CASE(32, 6)
  AERIS_SHORT_CASE(64, 1)
  AERIS_SHORT_CASE(64, 2)
  AERIS_SHORT_CASE(64, 3)
  AERIS_SHORT_CASE(64, 5)
  AERIS_SHORT_CASE(64, 6)
  AERIS_SHORT_CASE(128, 1)
  AERIS_SHORT_CASE(128, 2)
  AERIS_SHORT_CASE(128, 3)
  AERIS_SHORT_CASE(128, 4)
#undef AERIS_SHORT_CASE
  return -1;
}

}  // namespace aeris
