// Paged decode attention over a FlowKV pool, for gfx950 (MI355X).
//
// FlowKV (arXiv 2504.03775), section 3.3, restructures the KV pool to the
// block-major (B, L, 2, H) layout of Eq. 5 so a transfer moves few large
// ranges, and adapts the PagedAttention kernel to read it.  This is that
// consumer: the decode step of Eq. 2 -- one new query token per request
// attending to the request's cached K and V of one layer -- reading either
// layout through the request's block list.  Grouped KV heads: Hq query heads
// share Hkv KV heads, query head h reading KV head h / (Hq / Hkv).
//
// Decode attention reads every cached K and V element once and does about
// G flops per byte (G = Hq / Hkv query heads per KV head): it is HBM-bound,
// and the work per token is kept small enough that the loads stay the limit.
// Work split (flash-decoding style):
//   pass 1: one workgroup of four waves per (KV head, token split, request),
//           on the matrix cores for every head count (split_pass).
//   pass 2: one wave or workgroup per (query head, request) merges the
//           splits, several splits per thread in flight; not launched where
//           one split covers the longest request.
// The grid covers every split up to the longest request.  When the caller
// passes the lengths on the host they ride in the kernel arguments (the
// kLens instantiations): a split past its request's end then leaves before
// any memory access and writes nothing, and pass 2 reads only the
// request's own splits.  Otherwise the lengths come from device memory and
// such a split leaves an empty record for pass 2.
// Scores, weights and sums are float32 (a weight enters the matrix cores as
// three bfloat16 parts that hold all its 24 bits); exponentials are exp2 of
// scores scaled by log2(e).  K and V are bfloat16; the output is float32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "flowkv.h"
#include "flowkv_device.h"
#include "flowkv_status.h"

using flowkv::fail;
using flowkv::ok;

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) u32x4 gvec4;
typedef __attribute__((address_space(1))) u32x2 gvec2;
// float vectors of the workspace and the output, which are only 4-byte aligned
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Pass-1 workgroups: four waves (eight, a step's bytes being the same per
// wave, lost 2-50% at the same split: fewer workgroups to balance).
constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kTile = 32;                  // tokens per wave step
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLazy = 8.f;               // log2 of the largest unnormalised weight

struct AttnArgs {
  const char* base[FLOWKV_MAX_LAYERS];  // pool tensors (layer-major) or base[0]
  int64_t pool_blocks;
  int64_t chunk_bytes;                  // bs * Hkv * Dh * 2
  int64_t block_bytes;                  // 2 * L * chunk_bytes
  const uint16_t* q;                    // (n_req, Hq, Dh) bf16
  const int32_t* tables;                // (n_req, max_blocks)
  const int32_t* seq_lens;              // (n_req)
  float* out;                           // (n_req, Hq, Dh) f32
  float* ws;                            // the splits' records (record_sums, record_ml)
  int32_t layer, n_req, block_size, kv_heads, q_heads, max_blocks;
  int32_t split_tokens, max_splits, max_seq_len;
  float scale_log2;                     // scale * log2(e)
  // the requests' lengths, when the caller passed them on the host (the
  // kernels instantiated with kLens read these instead of seq_lens)
  int32_t lens[FLOWKV_ATTN_INLINE_LENS];
};
// The compiler appends 256 bytes of implicit arguments; the whole segment
// stays within 4 KiB.
static_assert(sizeof(AttnArgs) + 256 <= 4096, "kernel arguments must stay within 4 KiB");

// Tokens of a request that take part: its length, capped by its block list
// and by max_seq_len (which also bounds the workspace's split count).
__device__ __forceinline__ int clamp_len(const AttnArgs& a, int T) {
  const int by_table = a.max_blocks * a.block_size;
  T = T < by_table ? T : by_table;
  return T < a.max_seq_len ? T : a.max_seq_len;
}

// The workspace holds a record per (request, query head, split): the weighted
// V (Dh floats) of all records first, then all records' (reference max, sum).
// (With a record's Dh + 2 floats together, no 16-byte access to a weighted V
// was aligned but every second one.)
__device__ __forceinline__ int64_t record_at(const AttnArgs& a, int r, int h, int split) {
  return (int64_t(r) * a.q_heads + h) * a.max_splits + split;
}
__device__ __forceinline__ float* record_sums(const AttnArgs& a, int dh, int64_t rec) {
  return a.ws + rec * dh;
}
__device__ __forceinline__ f32x2u* record_ml(const AttnArgs& a, int dh, int64_t rec) {
  const int64_t n = int64_t(a.n_req) * a.q_heads * a.max_splits;
  return reinterpret_cast<f32x2u*>(a.ws + n * dh) + rec;
}

// Without the lengths in the arguments, a split at or past its request's end
// still leaves a record, an empty partial (max -inf, sum 0) for each of its
// kG query heads, so that the merge reads every split up to max_splits
// without the request's length.  Its weighted-V part is never written; the
// merge ignores it.  Where pass 1 writes the output itself, a request with no
// token gets zeros.
template <int kG, int kDh, bool kDirect>
__device__ __forceinline__ void write_past_end(const AttnArgs& a, int g, int split, int r,
                                               int tid) {
  if constexpr (kDirect) {
    for (int i = tid; i < kG * kDh; i += kThreads)
      a.out[(int64_t(r) * a.q_heads + g * kG) * kDh + i] = 0.f;
  } else if (tid < kG) {
    *record_ml(a, kDh, record_at(a, r, g * kG + tid, split)) = f32x2u{-INFINITY, 0.f};
  }
}

template <int kW> struct Words;
template <> struct Words<4> {
  typedef u32x4 T;
  static __device__ __forceinline__ T load_nt(const char* p) {
    return __builtin_nontemporal_load((const gvec4*)p);
  }
};
template <> struct Words<2> {
  typedef u32x2 T;
  static __device__ __forceinline__ T load_nt(const char* p) {
    return __builtin_nontemporal_load((const gvec2*)p);
  }
};

// Two words' upper halves (two floats truncated to bf16), `lo`'s in the lower half.
__device__ __forceinline__ uint32_t pair_hi(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}
// Two words' lower halves, `lo`'s in the lower half.
__device__ __forceinline__ uint32_t pair_lo(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// A float truncated to bf16.
__device__ __forceinline__ float hi_part(float x) {
  return __uint_as_float(__float_as_uint(x) & 0xffff0000u);
}

// The LDS of a pass-1 workgroup.
template <int kDh>
struct SplitLds {
  int64_t off[FLOWKV_ATTN_MAX_SPLIT];      // byte offset of a token's row in the pool
  // K's staging, a tile per wave; after the loop the waves' weighted sums
  alignas(16) uint8_t area[kWaves * kTile * kDh * 2];
  uint32_t dead[FLOWKV_ATTN_MAX_SPLIT / kTile];
  float m[kWaves][16], l[kWaves][16];
};

// Pass 1 on the matrix cores.  Each wave takes its own tiles of 32 tokens,
// four tiles apart; per tile:
//   - K and V rows arrive whole: 16 lanes read one token's head vector (Dh 64:
//     8 lanes for K, 16 of 8 bytes for V), so every instruction reads full
//     128-byte lines, and consecutive tokens: 4 rows a slot apart, of one block
//     but at a block's edge.  (Rows 8 tokens apart mostly lay in two blocks, which
//     in a block-major pool are megabytes apart: 1.2% slower on the 32-request
//     batch, 256.7 against 259.9 us.)  A lane of group q4 = lane / 16 holds V of
//     the tokens 4 e + q4 (e = 0..7), dims kT c16 .. + kT (c16 = lane % 16).
//   - K goes through the wave's LDS tile into the A operand, its 16-byte
//     pieces swizzled so that neither side conflicts.  (Loading the operand
//     straight from memory reads 64 bytes of 16 tokens per instruction: 4-12%
//     slower overall, 257.9 against 243.2 us on the 32-request batch.)
//   - S^T (32 tokens x 16 columns) = K Q^T by 16x16x32 MFMAs, row m of half gg
//     being token 16 gg + 4 (m % 4) + m / 4: a lane then holds, for one head, the
//     scores of exactly the eight tokens whose V it holds, in the order of the A
//     operand of P.V.  So P needs no exchange between lanes, and V's B operand
//     is a transpose inside the lane.  Each head has kRep columns (its number is
//     head_of(c16)), one for each part of its weights.
//   - online softmax: the reference max of a head moves only when some score
//     exceeds it by more than kLazy (log2 units), a wave-uniform branch that
//     is rarely taken after the first tile.
//   - P is cut into three bf16 parts by truncation, which hold its 24 bits
//     exactly, and the columns of a head carry one each: P.V is one MFMA per 16
//     dims, and each part has sums of its own, joined once per split (of four
//     columns the last is spare).  With 8 heads there are two columns and two
//     MFMAs: the second brings the third part to the second's sums.  (Three MFMAs
//     onto one sum rounded it three times as often.  Against 64 bits: 1.9e-7 for
//     2.3e-7 on the 32-request batch, 2.0e-7 for 2.6e-7 at 8 heads of 128, 1.6e-7
//     for 1.8e-7 at head_dim 64.)  The parts of a weight above zero are kept from
//     zero by 2^-133, bf16's smallest value, so that an infinite V gives what P V
//     gives and not 0 x inf; those of a zero weight are zero, so that no V is
//     large enough to add anything under it.
//   - the next tile's K loads are issued as soon as q.k has its operand, its V
//     loads after P.V; past the wave's last tile they read the split's first
//     row, which keeps their count static.
// What bounds it: HBM, and a CU's own rate.  A step's instructions are a fifth
// of the time its 16 KB take at 6 TB/s, whatever G is, so one form serves 1 to
// 8 query heads per KV head.  A CU alone draws about 40 bytes a nanosecond, with
// four waves or eight.  Registers (166 a lane at Dh 128) allow three workgroups
// per CU, at Dh 64 (94-96) four are asked for.  Both passes, against the form
// before this one (vector units up to 4 heads per KV head and at head_dim 64;
// events around graphs, one MI355X): 32 requests of 2,000-20,000 tokens, G 4,
// 255.9 us for 258.9; 48 of 30-1,500, 37.9 for 52.5; one of 13,000, 14.5 for
// 19.8; 16 x 32,000, G 8, one KV head, 45.9 for 49.5; head_dim 64, 24 of
// 300-6,000, G 2, 22.3 for 26.1.
//
// kDirect: one split covers the longest request, and this pass writes the
// output (a flag read at run time cost every other call 0.4 us).
template <int kDh, int kG, bool kLM, bool kLens, bool kDirect>
__device__ __forceinline__ void split_pass(const AttnArgs& a) {
  constexpr int kI = kDh / 32;                   // MFMA steps of K.q
  constexpr int kT = kDh / 16;                   // dims a lane owns in P.V
  constexpr int kVW = kT / 2;                    // V words per token and lane
  constexpr int kPc = kDh / 8;                   // 16-byte pieces of a K row
  constexpr int kKL = kTile * kPc / 64;          // K loads of a tile and lane
  constexpr int kRep = kG == 8 ? 2 : 4;          // columns of S, and rows of P, per head
  using VT = typename Words<kVW>::T;
  const int g = blockIdx.x, split = blockIdx.y, r = blockIdx.z;
  const int tid = threadIdx.x, ln = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar loop control
  const int q4 = ln >> 4, c16 = ln & 15;         // MFMA lane coordinates

  const int t0 = split * a.split_tokens;
  const int bs = a.block_size;
  // with the length in the arguments, a split past the request's end leaves
  // at once, before any memory access, and writes no record
  if constexpr (kLens && !kDirect)
    if (t0 >= clamp_len(a, a.lens[r])) return;
  if (t0 >= a.max_blocks * bs) {
    write_past_end<kG, kDh, kDirect>(a, g, split, r, tid);
    return;
  }
  // the byte offset of every token's row in the pool, staged once in LDS (of a
  // tile, token 4 e + q4 at 8 q4 + e); a token past the end or with a block
  // outside the pool reads the pool's first slot and has its bit set in its
  // tile's mask.  The block IDs are fetched without waiting for the request's
  // length.
  __shared__ SplitLds<kDh> lds;
  constexpr int kStage = FLOWKV_ATTN_MAX_SPLIT / kThreads;
  int32_t blk[kStage], slot[kStage];
#pragma unroll
  for (int i = 0; i < kStage; ++i) {
    const int x = tid + i * kThreads;
    if (x < a.split_tokens) {
      const uint32_t b = uint32_t(t0 + x) / uint32_t(bs);
      slot[i] = int32_t(uint32_t(t0 + x) - b * uint32_t(bs));
      blk[i] = a.tables[int64_t(r) * a.max_blocks +
                        (int32_t(b) < a.max_blocks ? int32_t(b) : a.max_blocks - 1)];
    }
  }
  // Q as the B operand of K.q: Q[head_of(c16)][32 i + 8 q4 .. + 8]
  auto head_of = [](int column) { return column / kRep % kG; };
  bf16x8 qb[kI];
#pragma unroll
  for (int i = 0; i < kI; ++i) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(
        a.q + (int64_t(r) * a.q_heads + g * kG + head_of(c16)) * kDh + 32 * i + 8 * q4);
    qb[i] = __builtin_bit_cast(bf16x8, w);
  }
  const int T = clamp_len(a, kLens ? a.lens[r] : a.seq_lens[r]);
  if (t0 >= T) {  // uniform: this split is past the request's end (no kLens)
    write_past_end<kG, kDh, kDirect>(a, g, split, r, tid);
    return;
  }
  const int n_tok = t0 + a.split_tokens < T ? a.split_tokens : T - t0;
  const int n_tiles = (n_tok + kTile - 1) / kTile;

  // pool addressing: K of (block b, slot) at kbase + b * bstride + slot *
  // sstride; V sits voff further
  const char* kbase;
  uint32_t bstride;
  int64_t voff;
  if constexpr (kLM) {
    kbase = a.base[a.layer];
    bstride = uint32_t(a.chunk_bytes);
    voff = a.pool_blocks * a.chunk_bytes;
  } else {
    kbase = a.base[0] + int64_t(a.layer) * 2 * a.chunk_bytes;
    bstride = uint32_t(a.block_bytes);
    voff = a.chunk_bytes;
  }
  const uint32_t sstride = uint32_t(a.kv_heads) * kDh * 2;
  kbase += g * kDh * 2;

#pragma unroll
  for (int i = 0; i < kStage; ++i) {
    const int x = tid + i * kThreads;
    const bool ok = x < n_tok && blk[i] >= 0 && blk[i] < a.pool_blocks;
    const uint64_t dead = __ballot(!ok);
    if (x < n_tiles * kTile) {
      lds.off[(x & -kTile) + (x & 3) * 8 + (x >> 2 & 7)] =
          ok ? int64_t(uint64_t(uint32_t(blk[i])) * bstride + uint32_t(slot[i]) * sstride) : 0;
      if (ln % kTile == 0) lds.dead[x / kTile] = uint32_t(dead >> ln);
    }
  }

  static_assert(sizeof(float) * kWaves * kG * kDh <= sizeof(lds.area), "merge area fits");
  u32x4* const s_k = reinterpret_cast<u32x4*>(lds.area + wave * (kTile * kDh * 2));

  f32x4 o[kT];
#pragma unroll
  for (int t = 0; t < kT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mref = -INFINITY, lsum = 0.f;            // of the column's head; this lane's tokens
  __syncthreads();

  // which part the column carries: what is taken off a weight before it
  const int part = c16 % kRep;
  const float off1 = part > 0 ? -1.f : 0.f, off2 = part > 1 ? -1.f : 0.f;
  u32x4 kw[kKL];
  VT vw[8];
  // K loads: lane ln takes piece kp of the tokens kt + e kStride, whose offsets
  // are at k_at + e kStride / 4
  constexpr int kStride = 64 / kPc;
  const int kt = ln / kPc, kp = ln % kPc;
  const int k_at = (kt & 3) * 8 + (kt >> 2);
  // a row's pieces are XORed with a number that differs among the 16 rows of
  // one operand read (at Dh 64, where two rows fill the banks, among the 8 pairs)
  auto swz = [](int token) { return (token * kPc >> 4) & (kPc - 1); };
  auto load_k = [&](int tile, bool real) {
#pragma unroll
    for (int e = 0; e < kKL; ++e)
      kw[e] = Words<4>::load_nt(kbase + 16 * kp +
                                lds.off[real ? tile * kTile + k_at + e * (kStride / 4) : 0]);
  };
  auto load_v = [&](int tile, bool real) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      vw[e] = Words<kVW>::load_nt(kbase + voff + c16 * (kVW * 4) +
                                  lds.off[real ? tile * kTile + 8 * q4 + e : 0]);
  };
  if (wave < n_tiles) {
    load_k(wave, true);
    load_v(wave, true);
  }
  for (int tile = wave; tile < n_tiles; tile += kWaves) {
    const bool more = tile + kWaves < n_tiles;
#pragma unroll
    for (int e = 0; e < kKL; ++e) {
      const int token = kt + e * kStride;
      s_k[token * kPc + (kp ^ swz(token))] = kw[e];
    }
    __builtin_amdgcn_wave_barrier();
    const int kr[2] = {4 * (c16 & 3) + (c16 >> 2), 16 + 4 * (c16 & 3) + (c16 >> 2)};
    bf16x8 ka[2][kI];
#pragma unroll
    for (int gg = 0; gg < 2; ++gg)
#pragma unroll
      for (int i = 0; i < kI; ++i)
        ka[gg][i] =
            __builtin_bit_cast(bf16x8, s_k[kr[gg] * kPc + ((4 * i + q4) ^ swz(kr[gg]))]);
    f32x4 s[2];
#pragma unroll
    for (int gg = 0; gg < 2; ++gg) {
      f32x4 si[kI];                              // joined as a tree: fewer roundings
#pragma unroll
      for (int i = 0; i < kI; ++i)
        si[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[gg][i], qb[i],
                                                        f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      if constexpr (kI == 4) s[gg] = (si[0] + si[1]) + (si[2] + si[3]);
      else s[gg] = si[0] + si[1];
    }
    __builtin_amdgcn_sched_barrier(0);
    load_k(tile + kWaves, more);
    __builtin_amdgcn_sched_barrier(0);
    // bit 4 e: the lane's token 4 e + q4 of this tile is dead
    uint32_t dead = __builtin_amdgcn_readfirstlane(lds.dead[tile]);
    const bool masked = dead != 0;               // uniform
    if (masked) {
      dead >>= q4;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (dead >> (4 * e) & 1) s[e >> 2][e & 3] = -INFINITY;
    }
    // scaled scores, rounded before the reference is taken off them (a fused
    // multiply-subtract would leave the largest token a weight other than 1)
    float p[8];
    {
#pragma clang fp contract(off)
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = s[e >> 2][e & 3] * a.scale_log2;
    }
    float mx = fmaxf(fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])),
                     fmaxf(fmaxf(p[4], p[5]), fmaxf(p[6], p[7])));
    if (__any(mx > mref + kLazy)) {              // also taken at the first live token
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      float c = 1.f;
      if (mx > mref + kLazy) {
        c = __builtin_amdgcn_exp2f(mref - mx);
        mref = mx;
      }
      lsum *= c;
#pragma unroll
      for (int j = 0; j < 4; j += kRep) {        // rows 4 q4 + j .. + kRep: one head
        const float cj = __shfl(c, 4 * q4 + j);
#pragma unroll
        for (int x = j; x < j + kRep; ++x)
#pragma unroll
          for (int t = 0; t < kT; ++t) o[t][x] *= cj;
      }
    }
    const float mu = mref == -INFINITY ? 0.f : mref;
    u32x4 pa, pb;                                // the column's part; with 8 heads, the third
    float lt[4];                                 // the tile's sum, in pairs
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma clang fp contract(off)
      uint32_t bw[2], ba[2], bb[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float w = __builtin_amdgcn_exp2f(p[2 * i + k] - mu);
        lt[i] = k == 0 ? w : lt[i] + w;
        bw[k] = __float_as_uint(w);
        if constexpr (kRep == 2) {
          const float r1 = w - hi_part(w);
          ba[k] = __float_as_uint(part > 0 ? r1 : w);
          bb[k] = __float_as_uint(part > 0 ? r1 - hi_part(r1) : 0.f);
        } else {
          const float r1 = fmaf(off1, hi_part(w), w);
          ba[k] = __float_as_uint(fmaf(off2, hi_part(r1), r1));
        }
      }
      const u16x2 one = {1, 1};
      const u16x2 least =
          __builtin_elementwise_min(__builtin_bit_cast(u16x2, pair_hi(bw[0], bw[1])), one);
      pa[i] = __builtin_bit_cast(
          uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, pair_hi(ba[0], ba[1])), least));
      if constexpr (kRep == 2)
        pb[i] = __builtin_bit_cast(
            uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, pair_hi(bb[0], bb[1])), least));
    }
    lsum += (lt[0] + lt[1]) + (lt[2] + lt[3]);
    // dead tokens' weight is 0, and 0 x a stale NaN would not be
    if (masked) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (dead >> (4 * e) & 1) vw[e] = VT{};
    }
    __builtin_amdgcn_sched_barrier(0);
    // two of the lane's dims at a time: their columns of the 8 tokens as B operands
#pragma unroll
    for (int m = 0; m < kVW; ++m) {
      u32x4 w[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        w[0][i] = pair_lo(vw[2 * i][m], vw[2 * i + 1][m]);
        w[1][i] = pair_hi(vw[2 * i][m], vw[2 * i + 1][m]);
      }
      auto add = [&](u32x4 p) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
          o[2 * m + h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, p), __builtin_bit_cast(bf16x8, w[h]), o[2 * m + h], 0, 0, 0);
      };
      add(pa);
      if constexpr (kRep == 2) add(pb);
    }
    __builtin_amdgcn_sched_barrier(0);
    load_v(tile + kWaves, more);
  }

  // merge the waves: per head a weight exp2(m_wave - M); a wave that saw no
  // token has m = -inf and weighs nothing
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  if (q4 == 0) {
    lds.m[wave][c16] = mref;
    lds.l[wave][c16] = lsum;
  }
  __syncthreads();  // every wave is past the loop: the area is free
  float* const s_o = reinterpret_cast<float*>(lds.area);   // [wave][head < kG][dim]
#pragma unroll
  for (int j = 0; j < 4; j += kRep)              // a head's parts, smallest first
    if (const int h = (4 * q4 + j) / kRep; h < kG) {
#pragma unroll
      for (int t = 0; t < kT; t += 4) {
        f32x4 x;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const f32x4 y = o[t + k];
          x[k] = kRep == 2 ? y[j + 1] + y[j] : y[2] + y[1] + y[0];
        }
        *reinterpret_cast<f32x4*>(&s_o[(wave * kG + h) * kDh + kT * c16 + t]) = x;
      }
    }
  __syncthreads();
  // kOut dims of one head per thread
  constexpr int kOut = kG * kDh > kThreads ? kG * kDh / kThreads : 1;
  typedef float OutLds __attribute__((ext_vector_type(kOut)));
  typedef float OutVec __attribute__((ext_vector_type(kOut), aligned(4)));
  if (tid * kOut >= kG * kDh) return;
  const int h = tid * kOut / kDh, d = tid * kOut % kDh;
  float M = -INFINITY, L = 0.f;
  OutVec A = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) M = fmaxf(M, lds.m[w][kRep * h]);
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float m = lds.m[w][kRep * h];
    const float wt = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
    const OutLds x = *reinterpret_cast<const OutLds*>(&s_o[(w * kG + h) * kDh + d]);
    L = fmaf(lds.l[w][kRep * h], wt, L);
#pragma unroll
    for (int k = 0; k < kOut; ++k) A[k] = fmaf(x[k], wt, A[k]);
  }
  if constexpr (kDirect) {
#pragma unroll
    for (int k = 0; k < kOut; ++k) A[k] = L == 0.f ? 0.f : A[k] / L;
    *reinterpret_cast<OutVec*>(a.out + (int64_t(r) * a.q_heads + g * kG + h) * kDh + d) = A;
  } else {
    const int64_t rec = record_at(a, r, g * kG + h, split);
    *reinterpret_cast<OutVec*>(record_sums(a, kDh, rec) + d) = A;
    if (d == 0) *record_ml(a, kDh, rec) = f32x2u{M, L};
  }
}

// (As the kernel's own body, split_pass came out 6% longer, and a 200-token
// call took 5.4 us for 5.2.)
// The waves per SIMD are an upper bound too: at Dh 64 the registers would
// let a fifth workgroup onto a CU while others are idle (24 requests of
// 300-6,000 tokens 25.8 us for 22.7).
template <int kDh, int kG, bool kLM, bool kLens, bool kDirect>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kDh == 64 ? 4 : 3, kDh == 64 ? 4 : 3)))
void decode_attn_split(const AttnArgs a) {
  split_pass<kDh, kG, kLM, kLens, kDirect>(a);
}

// Pass 2: the splits' records of one (query head, request), by one wave (up to
// kMergeChunk records per lane group; a workgroup then takes four heads) or by
// the four waves of a workgroup.  A group of Dh / 4 lanes takes a record, 4
// dims a lane, kMergeChunk records at once with no branch on their values (a
// split past the end re-reads split 0 and is masked), folded into a running
// (max, sum, weighted V) that is rescaled when its max rises; the groups then
// meet by lane exchanges, the waves in LDS.
// What bounds it: a launch's floor (about 3 us here) and one round of loads
// that come from HBM, since pass 1 wrote them on other XCDs.  The form before
// it took a float a lane and 16 records a thread however few there were: 48
// requests of up to 6 splits, 32 heads, 6.5 us against 3.9; 32 requests x 64
// heads x 16 splits at head_dim 64, 8.0 against 4.5; one request of 51 splits
// 4.6 against 4.0.
constexpr int kMergeThreads = 256;
constexpr int kMergeChunk = 4;

struct Running {
  float m, l;
  f32x4 v;
};

// Both parts' sums under the larger reference; a part that saw no token has
// m = -inf and weighs nothing.
__device__ __forceinline__ Running join(const Running& a, const Running& b) {
  Running r;
  r.m = fmaxf(a.m, b.m);
  const float wa = a.m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(a.m - r.m);
  const float wb = b.m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(b.m - r.m);
  r.l = a.l * wa + b.l * wb;
  r.v = a.v * wa + b.v * wb;
  return r;
}

template <int kDh, bool kLens, int kWavesPer>
__global__ __launch_bounds__(kMergeThreads) void decode_attn_merge(const AttnArgs a) {
  constexpr int kLanes = kDh / 4;                // lanes per record
  constexpr int kParts = 64 * kWavesPer / kLanes;
  const int r = blockIdx.y, ln = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = kWavesPer == 1 ? blockIdx.x * (kMergeThreads / 64) + wave : blockIdx.x;
  if (h >= a.q_heads) return;                    // (whole waves, and no barrier follows)
  const int tid = kWavesPer == 1 ? ln : threadIdx.x;
  const int d = 4 * (tid % kLanes), part = tid / kLanes;
  // records per (request, head); with the lengths in the arguments only the
  // request's own splits hold one
  int ns = a.max_splits;
  if constexpr (kLens) ns = (clamp_len(a, a.lens[r]) + a.split_tokens - 1) / a.split_tokens;
  const int64_t rec0 = record_at(a, r, h, 0);
  const float* sums = record_sums(a, kDh, rec0) + d;
  const f32x2u* ml = record_ml(a, kDh, rec0);
  Running x{-INFINITY, 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
  for (int x0 = part; x0 < ns; x0 += kParts * kMergeChunk) {
    // branch-free loads: a split past the end re-reads split 0 and is
    // masked; an empty record's weighted V (never written) is not used
    f32x2u m[kMergeChunk];
    f32x4u v[kMergeChunk];
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) {
      const int s = x0 + j * kParts < ns ? x0 + j * kParts : 0;
      m[j] = ml[s];
      v[j] = *reinterpret_cast<const f32x4u*>(sums + int64_t(s) * kDh);
    }
    float cm = x.m;
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) {
      if (x0 + j * kParts >= ns) m[j] = f32x2u{-INFINITY, 0.f};
      cm = fmaxf(cm, m[j][0]);
    }
    const float c = x.m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x.m - cm);
    x.l *= c;
    x.v *= c;
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) {
      // (a split whose scores are all NaN has a max of -inf, and a sum of NaN)
      const bool live = m[j][0] != -INFINITY || m[j][1] != 0.f;
      const float w = live ? __builtin_amdgcn_exp2f(m[j][0] - cm) : 0.f;
      x.l = live ? fmaf(m[j][1], w, x.l) : x.l;
#pragma unroll
      for (int k = 0; k < 4; ++k) x.v[k] = live ? fmaf(v[j][k], w, x.v[k]) : x.v[k];
    }
    x.m = cm;
  }
#pragma unroll
  for (int off = kLanes; off < 64; off *= 2) {
    Running y;
    y.m = __shfl_xor(x.m, off);
    y.l = __shfl_xor(x.l, off);
#pragma unroll
    for (int k = 0; k < 4; ++k) y.v[k] = __shfl_xor(x.v[k], off);
    x = join(x, y);
  }
  if constexpr (kWavesPer > 1) {
    __shared__ float s_ml[kWavesPer][2];
    __shared__ f32x4 s_v[kWavesPer][kLanes];
    if (ln < kLanes) s_v[wave][ln] = x.v;
    if (ln == 0) {
      s_ml[wave][0] = x.m;
      s_ml[wave][1] = x.l;
    }
    __syncthreads();
    if (threadIdx.x >= kLanes) return;
    x = Running{s_ml[0][0], s_ml[0][1], s_v[0][ln]};
#pragma unroll
    for (int w = 1; w < kWavesPer; ++w) x = join(x, Running{s_ml[w][0], s_ml[w][1], s_v[w][ln]});
  }
  if (part == 0) {
    f32x4u o;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = x.l == 0.f ? 0.f : x.v[k] / x.l;
    *reinterpret_cast<f32x4u*>(a.out + (int64_t(r) * a.q_heads + h) * kDh + d) = o;
  }
}

using SplitFn = void (*)(AttnArgs);

template <int D, bool LM, bool L, bool O>
SplitFn pick_group(int G) {
  switch (G) {
    case 1: return decode_attn_split<D, 1, LM, L, O>;
    case 2: return decode_attn_split<D, 2, LM, L, O>;
    case 4: return decode_attn_split<D, 4, LM, L, O>;
    default: return decode_attn_split<D, 8, LM, L, O>;
  }
}

template <bool L, bool O>
SplitFn pick_shape(int D, int G, bool lm) {
  if (D == 64) return lm ? pick_group<64, true, L, O>(G) : pick_group<64, false, L, O>(G);
  return lm ? pick_group<128, true, L, O>(G) : pick_group<128, false, L, O>(G);
}

template <bool L>
SplitFn pick_split_lens(int D, int G, bool lm, bool direct) {
  return direct ? pick_shape<L, true>(D, G, lm) : pick_shape<L, false>(D, G, lm);
}

SplitFn pick_split(int D, int G, bool lm, bool lens, bool direct) {
  return lens ? pick_split_lens<true>(D, G, lm, direct) : pick_split_lens<false>(D, G, lm, direct);
}

template <int D, bool L>
const void* pick_merge_waves(bool one) {
  return one ? reinterpret_cast<const void*>(decode_attn_merge<D, L, 1>)
             : reinterpret_cast<const void*>(decode_attn_merge<D, L, 4>);
}

const void* pick_merge(int D, bool lens, bool one) {
  if (D == 64) return lens ? pick_merge_waves<64, true>(one) : pick_merge_waves<64, false>(one);
  return lens ? pick_merge_waves<128, true>(one) : pick_merge_waves<128, false>(one);
}

// LDS that a launch of pass 1 asks for beyond the kernel's own, so that a CU
// takes no third workgroup where two per CU hold them all (`live`: with the
// lengths on the host the splits that do not leave at once, else all).  The
// dispatcher fills a CU as far as registers and LDS allow before every CU has
// its share: 342 workgroups of 24 requests on 2 KV heads took 26.4 us for 22.3,
// 356 of 31 requests 47.0 for 38.1, 360 at 8 heads 18.1 for 15.5; of 50 other
// calls of at most two per CU none was slower by more than the runs differ.
// With a third allowed beyond that, a limit of one less than fit cost up to 14%.
// No more workgroups than the smallest partition of the card has CUs are left as
// they are, without a lookup of the CU count (0.1 us of a call).
constexpr int64_t kFewestCus = 32;
constexpr int64_t kCuLds = 160 * 1024;
static_assert(sizeof(SplitLds<128>) <= kCuLds / 3, "two workgroups are spread by LDS alone");

unsigned spread_lds(int D, int64_t live, int64_t cus) {
  if (live <= kFewestCus || live > 2 * cus) return 0;
  return unsigned(kCuLds / 3 + 1 - (D == 64 ? sizeof(SplitLds<64>) : sizeof(SplitLds<128>)));
}

int32_t auto_split(int32_t n_req, int32_t max_seq_len) {
  for (int32_t s = FLOWKV_ATTN_MIN_AUTO_SPLIT; s < FLOWKV_ATTN_MAX_SPLIT; s *= 2)
    if (int64_t(n_req) * ((int64_t(max_seq_len) + s - 1) / s) <= FLOWKV_ATTN_AUTO_PAIRS) return s;
  return FLOWKV_ATTN_MAX_SPLIT;
}

int64_t ws_bytes(int32_t n_req, int32_t q_heads, int32_t head_dim, int32_t max_seq_len,
                 int32_t split_tokens) {
  const int64_t splits = (int64_t(max_seq_len) + split_tokens - 1) / split_tokens;
  return int64_t(n_req) * q_heads * splits * (head_dim + 2) * int64_t(sizeof(float));
}

}  // namespace

extern "C" int flowkv_decode_attention_split(int32_t n_req, int32_t max_seq_len,
                                             int32_t* split_tokens) {
  if (!split_tokens) return fail(FLOWKV_EINVAL, "NULL output");
  if (n_req < 0 || max_seq_len < 0) return fail(FLOWKV_EINVAL, "negative sizes");
  *split_tokens = auto_split(n_req, max_seq_len);
  return ok();
}

extern "C" int flowkv_decode_attention_workspace(int32_t n_req, int32_t q_heads,
                                                 int32_t head_dim, int32_t max_seq_len,
                                                 int32_t split_tokens, int64_t* bytes) {
  if (!bytes) return fail(FLOWKV_EINVAL, "NULL output");
  if (n_req < 0 || q_heads < 1 || head_dim < 1 || max_seq_len < 0)
    return fail(FLOWKV_EINVAL, "bad attention shape");
  if (split_tokens == 0) split_tokens = auto_split(n_req, max_seq_len);
  if (split_tokens < 1 || split_tokens > FLOWKV_ATTN_MAX_SPLIT)
    return fail(FLOWKV_EINVAL, "split_tokens %d: need 1..%d", split_tokens,
                FLOWKV_ATTN_MAX_SPLIT);
  *bytes = ws_bytes(n_req, q_heads, head_dim, max_seq_len, split_tokens);
  return ok();
}

namespace {

// Checks every argument, then enqueues both passes with `ws` (ws_cap bytes)
// as the workspace.  When `scratch_ws` is set, the workspace is the library's
// own device array (found after the checks, so a call rejected on its
// arguments makes no runtime call) and a short capacity is reported as such.
int launch_attention(const flowkv_pool* pool, int32_t layer, const void* q_dev, int32_t n_req,
                     int32_t q_heads, int32_t kv_heads, int32_t head_dim,
                     const int32_t* block_tables_dev, int32_t max_blocks,
                     const int32_t* seq_lens_dev, const int32_t* seq_lens_host,
                     int32_t max_seq_len, float scale, int32_t split_tokens, float* out_dev,
                     void* ws, int64_t ws_cap, bool scratch_ws, void* hip_stream);

}  // namespace

extern "C" int flowkv_decode_attention(const flowkv_pool* pool, int32_t layer,
                                       const void* q_dev, int32_t n_req, int32_t q_heads,
                                       int32_t kv_heads, int32_t head_dim,
                                       const int32_t* block_tables_dev, int32_t max_blocks,
                                       const int32_t* seq_lens_dev,
                                       const int32_t* seq_lens_host, int32_t max_seq_len,
                                       float scale, int32_t split_tokens, float* out_dev,
                                       void* workspace_dev, int64_t workspace_bytes,
                                       void* hip_stream) {
  return launch_attention(pool, layer, q_dev, n_req, q_heads, kv_heads, head_dim,
                          block_tables_dev, max_blocks, seq_lens_dev, seq_lens_host,
                          max_seq_len, scale, split_tokens, out_dev, workspace_dev,
                          workspace_bytes, false, hip_stream);
}

// ---- the variant that allocates nothing --------------------------------------
//
// Its partial results live in `scratch`, a file-scope device array: each GPU
// the library runs on holds its own copy for the life of the process.  In
// host code `scratch` names a host-side stand-in, not device memory; the
// device address of the current GPU's copy comes from hipGetSymbolAddress,
// looked up once per device on its first call and kept in g_scratch_addr.
// Nothing in the array needs to start at zero: pass 1 writes every split
// record the merge reads.  Calls that overlap on one GPU share the array and
// race.
static __device__ __align__(256) float scratch[FLOWKV_ATTN_SCRATCH_BYTES / sizeof(float)];
static_assert(FLOWKV_ATTN_SCRATCH_BYTES % 256 == 0, "scratch size in whole 256-byte units");

namespace {

constexpr int kMaxDevices = 64;

std::atomic<void*> g_scratch_addr[kMaxDevices];
std::mutex g_scratch_mu;

// Device address of the current GPU's copy of `scratch`.
int scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(FLOWKV_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(FLOWKV_EINVAL, "device %d: the scratch table holds devices 0..%d", dev,
                kMaxDevices - 1);
  void* p = g_scratch_addr[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    p = g_scratch_addr[dev].load(std::memory_order_relaxed);
    if (!p) {
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p)
        return fail(FLOWKV_EHIP, "scratch address on device %d: %s", dev,
                    hipGetErrorString(e));
      g_scratch_addr[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return FLOWKV_OK;
}

}  // namespace

extern "C" int flowkv_decode_attention_noalloc(const flowkv_pool* pool, int32_t layer,
                                               const void* q_dev, int32_t n_req,
                                               int32_t q_heads, int32_t kv_heads,
                                               int32_t head_dim,
                                               const int32_t* block_tables_dev,
                                               int32_t max_blocks, const int32_t* seq_lens_dev,
                                               const int32_t* seq_lens_host,
                                               int32_t max_seq_len, float scale,
                                               int32_t split_tokens, float* out_dev,
                                               void* hip_stream) {
  return launch_attention(pool, layer, q_dev, n_req, q_heads, kv_heads, head_dim,
                          block_tables_dev, max_blocks, seq_lens_dev, seq_lens_host,
                          max_seq_len, scale, split_tokens, out_dev, nullptr,
                          FLOWKV_ATTN_SCRATCH_BYTES, true, hip_stream);
}

namespace {

int launch_attention(const flowkv_pool* pool, int32_t layer, const void* q_dev, int32_t n_req,
                     int32_t q_heads, int32_t kv_heads, int32_t head_dim,
                     const int32_t* block_tables_dev, int32_t max_blocks,
                     const int32_t* seq_lens_dev, const int32_t* seq_lens_host,
                     int32_t max_seq_len, float scale, int32_t split_tokens, float* out_dev,
                     void* workspace_dev, int64_t workspace_bytes, bool scratch_ws,
                     void* hip_stream) {
  if (!pool) return fail(FLOWKV_EINVAL, "NULL pool");
  if (pool->layout != FLOWKV_LAYOUT_LAYER_MAJOR && pool->layout != FLOWKV_LAYOUT_BLOCK_MAJOR)
    return fail(FLOWKV_EINVAL, "unknown layout %d", pool->layout);
  if (pool->num_layers < 1 || pool->num_layers > FLOWKV_MAX_LAYERS || pool->num_blocks < 1 ||
      !pool->layer_base)
    return fail(FLOWKV_EINVAL, "bad pool descriptor");
  if (layer < 0 || layer >= pool->num_layers)
    return fail(FLOWKV_EINVAL, "layer %d outside the pool's %d layers", layer, pool->num_layers);
  if (head_dim != 64 && head_dim != 128)
    return fail(FLOWKV_EINVAL, "head_dim %d: need 64 or 128", head_dim);
  if (kv_heads < 1 || q_heads < 1 || q_heads % kv_heads)
    return fail(FLOWKV_EINVAL, "q_heads %d not a multiple of kv_heads %d", q_heads, kv_heads);
  const int G = q_heads / kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8)
    return fail(FLOWKV_EINVAL, "query heads per KV head %d: need 1, 2, 4 or 8", G);
  const int64_t per_token = int64_t(kv_heads) * head_dim * 2;
  if (pool->chunk_bytes <= 0 || pool->chunk_bytes % per_token)
    return fail(FLOWKV_EINVAL, "chunk_bytes %lld is not block_size x %d KV heads x %d bf16",
                (long long)pool->chunk_bytes, kv_heads, head_dim);
  const int64_t bs = pool->chunk_bytes / per_token;
  // the kernel forms block offsets in 32 bits: one block stride under 4 GiB
  const int64_t stride = pool->layout == FLOWKV_LAYOUT_LAYER_MAJOR
                             ? pool->chunk_bytes
                             : 2 * int64_t(pool->num_layers) * pool->chunk_bytes;
  if (stride >= (int64_t(1) << 32))
    return fail(FLOWKV_EINVAL, "block stride of %lld bytes: need under 4 GiB", (long long)stride);
  if (n_req < 0 || max_blocks < 0 || max_seq_len < 0)
    return fail(FLOWKV_EINVAL, "negative sizes");
  // token indices are 32-bit in the kernels: a table row addresses at most
  // 2^31 - 1 tokens
  if (int64_t(max_blocks) * bs > INT32_MAX)
    return fail(FLOWKV_EINVAL, "max_blocks %d x block_size %lld tokens: need at most 2^31 - 1",
                max_blocks, (long long)bs);
  if (split_tokens == 0) split_tokens = auto_split(n_req, max_seq_len);
  if (split_tokens < 1 || split_tokens > FLOWKV_ATTN_MAX_SPLIT)
    return fail(FLOWKV_EINVAL, "split_tokens %d: need 1..%d", split_tokens,
                FLOWKV_ATTN_MAX_SPLIT);
  if (!(scale > 0.f) || !std::isfinite(scale)) return fail(FLOWKV_EINVAL, "bad scale");
  if (n_req == 0) return ok();
  const int64_t need = ws_bytes(n_req, q_heads, head_dim, max_seq_len, split_tokens);
  // (a workspace of 0 bytes, when max_seq_len is 0, may be NULL)
  // lengths from the host ride in the kernel arguments (then the device
  // copy is not read)
  const bool lens = seq_lens_host && n_req <= FLOWKV_ATTN_INLINE_LENS;
  if (!q_dev || !block_tables_dev || (!seq_lens_dev && !lens) || !out_dev ||
      (!scratch_ws && !workspace_dev && need > 0))
    return fail(FLOWKV_EINVAL, "NULL device pointer");
  if (workspace_bytes < need) {
    if (scratch_ws)
      return fail(FLOWKV_ECAP,
                  "%lld bytes of partial results needed, the library's scratch holds %lld "
                  "(fewer requests or query heads per call, or a longer split)",
                  (long long)need, (long long)workspace_bytes);
    return fail(FLOWKV_ECAP, "workspace of %lld bytes, %lld needed", (long long)workspace_bytes,
                (long long)need);
  }
  if (reinterpret_cast<uintptr_t>(q_dev) % 16)
    return fail(FLOWKV_EINVAL, "query not 16-byte aligned");
  // the launch grids put requests and splits on dimensions limited to 65,535
  const int64_t splits = (int64_t(max_seq_len) + split_tokens - 1) / split_tokens;
  if (n_req > 65535 || splits > 65535)
    return fail(FLOWKV_EINVAL, "%d requests, %lld splits: each must be at most 65535 per call",
                n_req, (long long)splits);
  const bool lm = pool->layout == FLOWKV_LAYOUT_LAYER_MAJOR;
  const int nbase = lm ? pool->num_layers : 1;
  AttnArgs a{};
  for (int i = 0; i < nbase; ++i) {
    if (!pool->layer_base[i] || reinterpret_cast<uintptr_t>(pool->layer_base[i]) % 16)
      return fail(FLOWKV_EINVAL, "pool base pointer %d NULL or not 16-byte aligned", i);
    a.base[i] = static_cast<const char*>(pool->layer_base[i]);
  }
  if (scratch_ws && need > 0) {
    const int rc = scratch_address(&workspace_dev);
    if (rc) return rc;
  }
  a.pool_blocks = pool->num_blocks;
  a.chunk_bytes = pool->chunk_bytes;
  a.block_bytes = 2 * int64_t(pool->num_layers) * pool->chunk_bytes;
  a.q = static_cast<const uint16_t*>(q_dev);
  a.tables = block_tables_dev;
  a.seq_lens = seq_lens_dev;
  a.out = out_dev;
  a.ws = static_cast<float*>(workspace_dev);
  a.layer = layer;
  a.n_req = n_req;
  a.block_size = int32_t(bs);
  a.kv_heads = kv_heads;
  a.q_heads = q_heads;
  a.max_blocks = max_blocks;
  a.split_tokens = split_tokens;
  a.max_splits = int32_t(splits);
  a.max_seq_len = max_seq_len;
  a.scale_log2 = scale * kLog2e;
  // a call whose longest request is one split needs no merge: pass 1 divides
  // and writes the output, which saves a launch (one request of 200 tokens
  // 7.5 against 5.0 us, 64 of 100 at 8 heads per KV head 13.2 against 9.4)
  const bool direct = a.max_splits == 1;
  int64_t live = splits * n_req * kv_heads;
  if (lens) {
    live = 0;
    for (int32_t i = 0; i < n_req; ++i) {
      a.lens[i] = seq_lens_host[i];
      const int64_t T = std::min(std::max(a.lens[i], 0), max_seq_len);
      live += (T + split_tokens - 1) / split_tokens * kv_heads;
    }
  }
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  void* args[] = {&a};
  hipError_t e = hipSuccess;
  if (a.max_splits > 0) {
    int cus = 0;
    if (live > kFewestCus) {
      const int rc = flowkv::cu_count(&cus);
      if (rc) return rc;
    }
    SplitFn fn = pick_split(head_dim, G, lm, lens, direct);
    e = hipLaunchKernel(reinterpret_cast<const void*>(fn),
                        dim3(unsigned(kv_heads), unsigned(a.max_splits), unsigned(n_req)),
                        dim3(kThreads), args, spread_lds(head_dim, live, cus), st);
  }
  if (e == hipSuccess && !direct) {
    // one wave per (query head, request) where its lane groups hold every
    // record at once, a workgroup's four waves above
    const bool one = a.max_splits <= kMergeChunk * 64 * 4 / head_dim;
    e = hipLaunchKernel(pick_merge(head_dim, lens, one),
                        dim3(unsigned(one ? (q_heads + 3) / 4 : q_heads), unsigned(n_req)),
                        dim3(kMergeThreads), args, 0, st);
  }
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) return fail(FLOWKV_EHIP, "attention launch: %s", hipGetErrorString(e));
  return ok();
}

}  // namespace
