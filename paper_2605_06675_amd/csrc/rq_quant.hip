// Quantize + pack kernels (KIVI-style, QuaRot-style and plain per-token
// symmetric RTN) and the residual window append.  One wave quantizes one 32-token block of one
// (batch entry, kv-head, K|V) unit; the unit's bit-width and code region come
// from the per-layer table in the kernel arguments.
//
// The block's rows are copied straight to LDS.  KIVI's group statistics run
// along one axis of the block and packing along the other (keys: statistics
// per channel over the 32 tokens, chunks of 32 channels per token; values: the
// reverse), so each phase reads the rows or columns it needs from LDS and
// every code goes straight into its packed word.
#include "rq_device.h"
#include "rq_internal.h"
#include "rq_ring.h"

namespace rq {

namespace {

constexpr int kWave = 64;

__device__ __forceinline__ int pair_pos(int j) {
  return j < 16 ? 2 * j : 2 * (j - 16) + 1;
}

struct BlockId {
  int blk, h, b, kind;
};

// The block of a workgroup (see set_grid).
__device__ __forceinline__ BlockId block_id(const QuantLaunch& a) {
  int blk = blockIdx.x, y = blockIdx.y, b = blockIdx.z;
  if (a.ring_fused == kRingFirst) {
    // the first blocks of all units start first: their waves have the window
    // to copy as well (11 x 8 units of 64 blocks: 29.0 us with them in place)
    const unsigned ys = a.H * a.kind_n, units = ys * a.B;
    const unsigned i = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const unsigned rest = a.nblk > 1 ? a.nblk - 1 : 1, j = i - units;
    const unsigned unit = i < units ? i : j / rest;
    blk = i < units ? 0 : 1 + j - unit * rest;
    if (a.by_batch) {
      b = unit / ys;
      y = unit - b * ys;
    } else {
      y = unit / (unsigned)a.B;
      b = unit - y * a.B;
    }
  } else if (!a.by_batch) {
    b = blockIdx.x / (unsigned)a.nblk;
    blk -= b * a.nblk;
  }
  if (a.by_batch) {
    const int k = y >= a.H;
    return {a.blk0 + blk, y - k * a.H, b, a.kind_lo + k};
  }
  const int both = a.kind_n == 2;
  return {a.blk0 + blk, y >> both, b, a.kind_lo + (both ? y & 1 : 0)};
}

// ---------------------------------------------------------------- staging

// A block's rows go to LDS as they lie in memory (whole rows per instruction),
// 16-byte piece s of token t in slot s ^ (t % 8) of the row: the 16 lanes of a
// 16-byte read's turn then take all banks wherever they read one piece of
// eight tokens (two pieces apart by 8) or four pieces of four tokens.
constexpr int kRow = kD / 2;                 // dwords of a staged token
constexpr int kPass = 16 * kRow;             // dwords of 16 tokens
__device__ __forceinline__ int slot(int t, int piece) {     // dword of the piece
  return t * kRow + 4 * (piece ^ (t & 7));
}

// 32 consecutive rows into LDS, the first 16 tokens by the first four of eight
// copies.  AUX: cache policy.
template <int AUX>
__device__ __forceinline__ void copy_rows(const uint16_t* rows, int lane, uint32_t* sm) {
  const int g = lane >> 4, p = (lane & 15) ^ g;          // of token 4 j + g
  const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(rows), 0, kChunk * kD * 2, 0x00020000);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void*)(sm + 4 * kRow * j), 16,
                                             256 * g + 16 * (p ^ (j & 1 ? 4 : 0)), 1024 * j, 0,
                                             AUX);
}

// The block's rows into LDS; through registers where they don't lie in one
// piece (partly in the window, or in slots that wrap) or not at a multiple of
// the copies' 16 bytes.
__device__ __forceinline__ void stage_rows(const QuantLaunch& a, int b, int h, int kind, int t0,
                                           int lane, uint32_t* sm) {
  const uint16_t* in = (kind ? a.v : a.k) + (size_t)(b * a.H + h) * a.n_new * kD;
  if (t0 >= a.n_past && lds_copy_aligned(in)) {          // the same for the wave
    in += (size_t)(t0 - a.n_past) * kD;
    if (a.stream) copy_rows<2 /* NT */>(in, lane, sm);
    else copy_rows<0>(in, lane, sm);
    return;
  }
  // (slots by one division: with one a row, eight a wave, and rows through
  // registers a decode step's block, whose launch is one latency after
  // another, took QuaRot 6.2 us, so 5.6, RTN 5.1 and 4.5, KIVI 5.5 and 4.9)
  const int cap = a.R + kChunk, s0 = t0 % cap;
  const uint16_t* ring = a.resid + (((size_t)b * a.H + h) * 2 + kind) * cap * kD;
  const uint16_t* old = ring + (size_t)s0 * kD;
  if (t0 + kChunk <= a.n_past && s0 + kChunk <= cap && lds_copy_aligned(old)) {
    copy_rows<0>(old, lane, sm);
    return;
  }
  u4 x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int i = 4 * j + (lane >> 4), s = s0 + i;
    const uint16_t* row = t0 + i >= a.n_past ? in + (size_t)(t0 + i - a.n_past) * kD
                                             : ring + (size_t)(s < cap ? s : s - cap) * kD;
    x[j] = gptr(reinterpret_cast<const u4*>(row))[(lane & 15) ^ (lane >> 4) ^ (j & 1 ? 4 : 0)];
  }
#pragma unroll
  for (int j = 0; j < 8; ++j)
    *reinterpret_cast<u4*>(sm + 4 * kRow * j + 4 * lane) = x[j];
}

// Until at most N of the wave's copies are under way (the compiler does not
// track the LDS they write).
template <int N>
__device__ __forceinline__ void wait_rows() {
  static_assert(N < 16, "low bits of the count");
  __builtin_amdgcn_s_waitcnt(N | (7 << 4));      // and all LDS operations
  asm volatile("" ::: "memory");
}

// The launch's window rows that any wave may copy.
__device__ __forceinline__ void copy_any(const QuantLaunch& a, int lane) {
  copy_window(a.ring, (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x,
              gridDim.x * gridDim.y * gridDim.z, lane);
}

// The launch's window rows (called when the wave's own rows are staged).
__device__ __forceinline__ void copy_ring(const QuantLaunch& a, const BlockId& id, int lane) {
  if (a.ring_fused == kRingAny)
    copy_any(a, lane);
  else if (a.ring_fused == kRingFirst && id.blk == a.blk0)
    copy_unit_window(a.ring, id.b, id.h, id.kind, lane);
}

// ------------------------------------------------------------- KIVI (LDS)
// One wave a block: no barrier is needed, as a wave's LDS operations complete
// in issue order.  Memory bounds this kernel, so what counts is the bytes in
// flight: 16 waves a CU with 8 KB each (LDS bounds them: 9.6 KB a wave), a new
// wave's copies starting as soon as one ends.  Llama-3-8B layer, 16 x 8 x 8192
// tokens at 2.5 bits: 128 us with 12 persistent waves a CU that loaded the next
// block into registers, 108 us so (6.1 TB/s of rows, codes and metadata).
constexpr int kTabE = 34;                 // float2 entries per table row

struct KiviSmem {
  uint32_t x[kChunk * kRow];              // the rows, pieces as slot() places them
  float2 tab[4 * kTabE];                  // (zero, 1/scale): K [chunk][channel],
                                          // V [group][token]
  uint16_t meta[256];                     // the block's metadata (512 B)
};

template <int BF16>
__device__ __forceinline__ float lo16(uint32_t w) {
  if (BF16) return __uint_as_float(w << 16);
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu));
}
template <int BF16>
__device__ __forceinline__ float hi16(uint32_t w) {
  if (BF16) return __uint_as_float(w & 0xffff0000u);
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
}

// Group bounds of finite inputs (minimum/maximum map to the three-input
// instructions without canonicalising every operand).
__device__ __forceinline__ float vmin(float a, float b) {
  return __builtin_elementwise_minimum(a, b);
}
__device__ __forceinline__ float vmax(float a, float b) {
  return __builtin_elementwise_maximum(a, b);
}

constexpr uint32_t kMagicBits = 0x4B000000u;   // the float 2^23

// Code of x in the low bits of a float: the clamped quotient plus 2^23 is
// rounded by the fp32 add to the nearest integer, ties to even (the
// quotient lies in [0, 2^b - 1]), leaving rint(quotient) in the low
// mantissa bits under the constant field kMagicBits.
template <int B>
__device__ __forceinline__ uint32_t kivi_code_bits(float x, float zf, float inv) {
  float r = (x - zf) * inv;               // two roundings: fp-contract is off
  r = __builtin_amdgcn_fmed3f(r, 0.0f, (float)((1 << B) - 1));
  return __float_as_uint(r + 8388608.0f);
}

// Packed words of one chunk, built by adding each code's fields at their
// bit positions.  A code arrives as kMagicBits + code; the fields of a plane
// that reaches the top bit are added as (bits >> shift), which carries the
// constant kMagicBits >> shift along, and lower planes are extracted
// exactly.  Fields never overlap, so the sum equals the OR of the fields
// plus a compile-time constant per word, removed by finish().  A three-bit
// code is one field; its part that crosses into the next word is
// (bits >> k), k <= 2, which is (kMagicBits >> k) + (code >> k) because the
// low 24 bits of kMagicBits are zero.
template <int B> struct ChunkAcc {
  uint32_t w[B];
  uint32_t bias[B];

  __device__ __forceinline__ void init() {
#pragma unroll
    for (int i = 0; i < B; ++i) w[i] = 0, bias[i] = 0;
  }
  // code i of the chunk (0..31, constant after unrolling)
  __device__ __forceinline__ void add(int i, uint32_t cb) {
    if constexpr (B == 3) {
      const int pos = stream3_pos(i), word = pos >> 5, bit = pos & 31;
      w[word] += cb << bit;
      bias[word] += kMagicBits << bit;
      if (bit > 29) {
        w[word + 1] += cb >> (32 - bit);
        bias[word + 1] += kMagicBits >> (32 - bit);
      }
      return;
    } else {
      int word = 0, shift = 0;
#pragma unroll
      for (int p = 0; p < Planes<B>::n; ++p) {
        const int wd = Planes<B>::w[p];
        const int per = 16 / wd;
        const int j = i & 15, d = j / per, k = j % per;
        const int pos = k * wd + (i >= 16 ? 16 : 0);
        if (shift + wd == B) {
          w[word + d] += (cb >> shift) << pos;
          bias[word + d] += (kMagicBits >> shift) << pos;
        } else {
          w[word + d] += __builtin_amdgcn_ubfe(cb, shift, wd) << pos;
        }
        word += wd;
        shift += wd;
      }
    }
  }
  __device__ __forceinline__ void finish() {
#pragma unroll
    for (int i = 0; i < B; ++i) w[i] -= bias[i];
  }
};

// Code and metadata stores are non-temporal: written once per call and
// read by later calls, they need not stay in the L2 (whose dirty lines the
// end of the launch would otherwise write back).
template <int B>
__device__ __forceinline__ void store_chunk(uint32_t* dst, const uint32_t* w) {
  RQ_GLOBAL uint32_t* g = gptr(dst);
#pragma unroll
  for (int i = 0; i < B; ++i) __builtin_nontemporal_store(w[i], g + i);
}

// Metadata of the block, staged in LDS, to its 512-byte slot.
__device__ __forceinline__ void store_meta(const QuantLaunch& a, const KiviSmem& sm,
                                           const BlockId& id, int lane) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  const int nblk_cap = a.cap / kChunk;
  RQ_GLOBAL u2* m = gptr(reinterpret_cast<u2*>(
      a.meta + meta_unit_offset(a.family, id.h, id.kind, id.b, a.B, nblk_cap) +
      (size_t)id.blk * kMetaBlockKivi));
  __builtin_nontemporal_store(reinterpret_cast<const u2*>(sm.meta)[lane], m + lane);
}

// Keys: scale and zero per channel over the block's 32 tokens; chunk q of
// token t holds channels 32q .. 32q + 31.
template <int BF16, int B>
__device__ __forceinline__ void kivi_keys_lds(const QuantLaunch& a, KiviSmem& sm,
                                              const BlockId& id, int lane) {
  // statistics: lane -> channels 2 lane, 2 lane + 1
  float mn0 = INFINITY, mx0 = -INFINITY, mn1 = INFINITY, mx1 = -INFINITY;
#pragma unroll
  for (int t = 0; t < kChunk; ++t) {
    const uint32_t w = sm.x[t * kRow + (lane ^ (4 * (t & 7)))];
    const float x0 = lo16<BF16>(w), x1 = hi16<BF16>(w);
    mn0 = vmin(mn0, x0);
    mx0 = vmax(mx0, x0);
    mn1 = vmin(mn1, x1);
    mx1 = vmax(mx1, x1);
  }
  const float qmax = (float)((1 << B) - 1);
  const AsymParams p0 = asym_params(mn0, mx0, qmax);
  const AsymParams p1 = asym_params(mn1, mx1, qmax);
  {
    const int q = lane >> 4, j = 2 * (lane & 15);
    *reinterpret_cast<float4*>(&sm.tab[q * kTabE + j]) =
        make_float4(p0.zf, p0.inv, p1.zf, p1.inv);
    sm.meta[q * 64 + pair_pos(j)] = p0.s16;
    sm.meta[q * 64 + pair_pos(j + 1)] = p1.s16;
    sm.meta[q * 64 + 32 + pair_pos(j)] = p0.z16;
    sm.meta[q * 64 + 32 + pair_pos(j + 1)] = p1.z16;
  }
  __builtin_amdgcn_wave_barrier();
  store_meta(a, sm, id, lane);
  // packing: lane -> chunk q of tokens ta and ta + 16, one token at a time
  // (the table is read twice; holding both tokens' rows costs registers)
  const int q = lane & 3, ta = lane >> 2;
  uint32_t* region = reinterpret_cast<uint32_t*>(a.codes + a.tab.code_off[id.h][0]);
  const int t0 = id.blk * kChunk;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    ChunkAcc<B> acc;
    acc.init();
    const int t = ta + 16 * u;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      __builtin_amdgcn_sched_barrier(0);
      float zf[16], inv[16];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float4 e = *reinterpret_cast<const float4*>(
            &sm.tab[q * kTabE + 16 * half + 2 * i]);
        zf[2 * i] = e.x;
        inv[2 * i] = e.y;
        zf[2 * i + 1] = e.z;
        inv[2 * i + 1] = e.w;
      }
      const u4 d0 = *reinterpret_cast<const u4*>(&sm.x[slot(t, 4 * q + 2 * half)]);
      const u4 d1 = *reinterpret_cast<const u4*>(&sm.x[slot(t, 4 * q + 2 * half + 1)]);
      const uint32_t w[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = 16 * half + 2 * k;
        acc.add(i, kivi_code_bits<B>(lo16<BF16>(w[k]), zf[2 * k], inv[2 * k]));
        acc.add(i + 1, kivi_code_bits<B>(hi16<BF16>(w[k]), zf[2 * k + 1], inv[2 * k + 1]));
      }
    }
    acc.finish();
    const size_t tok = (size_t)id.b * a.cap + t0 + t;
    store_chunk<B>(region + (tok * 4 + q) * B, acc.w);
  }
}

// Values: scale and zero per token over each group of 32 channels; chunk c
// of the block holds channel c over its 32 tokens.
template <int BF16, int B>
__device__ __forceinline__ void kivi_values_lds(const QuantLaunch& a, KiviSmem& sm,
                                                const BlockId& id, int lane) {
  const float qmax = (float)((1 << B) - 1);
  {
    // statistics: lane -> token t, groups 2 hb and 2 hb + 1
    const int t = lane >> 1, hb = lane & 1;
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2) {
      const int g = 2 * hb + g2;
      float mn = INFINITY, mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const u4 d = *reinterpret_cast<const u4*>(&sm.x[slot(t, 4 * g + i)]);
        const uint32_t w[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x0 = lo16<BF16>(w[e]), x1 = hi16<BF16>(w[e]);
          mn = vmin(mn, vmin(x0, x1));
          mx = vmax(mx, vmax(x0, x1));
        }
      }
      const AsymParams p = asym_params(mn, mx, qmax);
      sm.tab[g * kTabE + t] = make_float2(p.zf, p.inv);
      sm.meta[g * 64 + pair_pos(t)] = p.s16;
      sm.meta[g * 64 + 32 + pair_pos(t)] = p.z16;
    }
  }
  __builtin_amdgcn_wave_barrier();
  store_meta(a, sm, id, lane);
  // packing: lane -> channels 2 lane, 2 lane + 1 (group lane / 16)
  const int g = lane >> 4;
  ChunkAcc<B> acc0, acc1;
  acc0.init();
  acc1.init();
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __builtin_amdgcn_sched_barrier(0);
    float zf[16], inv[16];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float4 e = *reinterpret_cast<const float4*>(
          &sm.tab[g * kTabE + 16 * half + 2 * i]);
      zf[2 * i] = e.x;
      inv[2 * i] = e.y;
      zf[2 * i + 1] = e.z;
      inv[2 * i + 1] = e.w;
    }
#pragma unroll
    for (int tt = 0; tt < 16; ++tt) {
      const int t = 16 * half + tt;
      const uint32_t w = sm.x[t * kRow + (lane ^ (4 * (t & 7)))];
      acc0.add(t, kivi_code_bits<B>(lo16<BF16>(w), zf[tt], inv[tt]));
      acc1.add(t, kivi_code_bits<B>(hi16<BF16>(w), zf[tt], inv[tt]));
    }
  }
  acc0.finish();
  acc1.finish();
  const int nblk_cap = a.cap / kChunk;
  uint32_t* dst = reinterpret_cast<uint32_t*>(a.codes + a.tab.code_off[id.h][1]) +
                  (((size_t)id.b * nblk_cap + id.blk) * kD + 2 * lane) * B;
  store_chunk<B>(dst, acc0.w);
  store_chunk<B>(dst + B, acc1.w);
}

template <int BF16, int MAXB>
__device__ __forceinline__ void kivi_block(const QuantLaunch& a, KiviSmem& sm,
                                           const BlockId& id, int lane) {
  const int bits = kernarg_byte(&a.tab.bits[0][0], 2 * id.h + id.kind);
#define RQ_KIVI_CASE(NB)                                          \
  case NB:                                                        \
    if (NB <= MAXB) {                                             \
      if (id.kind == 0)                                           \
        kivi_keys_lds<BF16, NB>(a, sm, id, lane);                 \
      else                                                        \
        kivi_values_lds<BF16, NB>(a, sm, id, lane);               \
    }                                                             \
    break;
  switch (bits) {
    RQ_KIVI_CASE(1)
    RQ_KIVI_CASE(2)
    RQ_KIVI_CASE(3)
    RQ_KIVI_CASE(4)
    RQ_KIVI_CASE(5)
    RQ_KIVI_CASE(6)
    RQ_KIVI_CASE(7)
    RQ_KIVI_CASE(8)
    default: break;
  }
#undef RQ_KIVI_CASE
}

// MAXB: the widest bit-width of the launch (4 or 8: up to 4 the code paths fit
// the 128 registers that four waves a SIMD leave)
template <int BF16, int MAXB>
__global__ void __launch_bounds__(kWave, MAXB <= 4 ? 4 : 3)
kivi_quant_kernel(QuantLaunch a) {
  __shared__ __attribute__((aligned(16))) KiviSmem sm;
  const int lane = threadIdx.x;
  const BlockId id = block_id(a);
  stage_rows(a, id.b, id.h, id.kind, id.blk * kChunk, lane, sm.x);
  wait_rows<0>();
  kivi_block<BF16, MAXB>(a, sm, id, lane);
  copy_ring(a, id, lane);
}

// ------------------------------------------------------- QuaRot and RTN
// Per-token symmetric quantization over the token's 128 channels; QuaRot
// (ROT = 1) first applies the orthonormal Hadamard rotation, RTN (ROT = 0)
// quantizes the vector as it is.
//
// One wave a block, in two passes of 16 tokens.  Lane -> token 16 p + lane / 4
// and quarter q = lane % 4, which is exactly packed chunk q of the token.  The
// block's rows go to LDS, each lane then reads its quarter.
//
// Vector instructions bound this kernel (Qwen3-8B layer, 8 x 8 x 32768 tokens,
// QuaRot at 4 bits: 265 us with the instruction count at 266 us of issue), then
// memory.  Writing the lane-crossing butterflies as one instruction, leaving
// the clamp out where the scale shows that it does nothing, one copy of the
// rotation for all widths and a transpose of code bytes by 16 dword reads in
// place of 64 byte reads: 233 us; whole-row copies to LDS with the loads' 32
// registers freed: 228 us (5.9 TB/s of rows, codes and metadata).
constexpr int kSymCodes = kPass + 32;        // from pass 0's code bytes to pass 1's:
                                             // half the banks apart

__device__ __forceinline__ float dpp_xor1(float v) {
  // quad_perm [1,0,3,2]: exchange with lane ^ 1
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF,
                                      0xF, true));
}

__device__ __forceinline__ float dpp_xor2(float v) {
  // quad_perm [2,3,0,1]: exchange with lane ^ 2
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF,
                                      0xF, true));
}

// v[i] + k * v[i] of lane ^ 1, then v[i] + k2 * v[i] of lane ^ 2.  (Written
// out: the compiler keeps a move for every DPP operand.  Such an operand is
// read at the earliest two instructions after it was written.)
__device__ __forceinline__ void butterfly_quad(float v[8], float k1, float k2) {
#define RQ_ST(CTRL, K)                                                                     \
  "v_fmac_f32_dpp %0, %0, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"      \
  "v_fmac_f32_dpp %1, %1, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"      \
  "v_fmac_f32_dpp %2, %2, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"      \
  "v_fmac_f32_dpp %3, %3, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"      \
  "v_fmac_f32_dpp %4, %4, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"      \
  "v_fmac_f32_dpp %5, %5, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"      \
  "v_fmac_f32_dpp %6, %6, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"      \
  "v_fmac_f32_dpp %7, %7, " K " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
  asm("s_nop 1\n\t" RQ_ST("quad_perm:[1,0,3,2]", "%8") RQ_ST("quad_perm:[2,3,0,1]", "%9")
      : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]),
        "+v"(v[7])
      : "v"(k1), "v"(k2));
#undef RQ_ST
}

// The rotation of a token held by a quad of lanes, this lane's quarter in v.
// The butterflies keep their order (stride 1 .. 16 inside the lane, then 32
// and 64 with lanes q ^ 1 and q ^ 2), so every value is the one that the
// definition computes.  The upper lane of a pair takes other - own, the
// lower one own + other: the caller has negated the inputs of the quarters
// q = 1 and 2, which is exact and makes each of the two stages one fma with
// a factor +-1 (the same single rounding of the same exact sum).
__device__ __forceinline__ void rotate_quarter(float v[32], int q) {
#pragma unroll
  for (int hh = 1; hh < 32; hh *= 2)
#pragma unroll
    for (int i = 0; i < 32; ++i)
      if ((i & hh) == 0) {
        const float x = v[i], y = v[i + hh];
        v[i] = x + y;
        v[i + hh] = x - y;
      }
  const float k1 = (q & 1) ? 1.0f : -1.0f, k2 = (q & 2) ? 1.0f : -1.0f;
#pragma unroll
  for (int i = 0; i < 32; i += 8) butterfly_quad(v + i, k1, k2);
  const float c = 0.08838834764831845f;  // fp32 nearest to 1/sqrt(128)
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = v[i] * c;
}

// The largest magnitude of a token.  NAN_OUT: a NaN gives NaN, else it does
// not count.
template <bool NAN_OUT>
__device__ __forceinline__ float quad_amax(const float v[32]) {
  if constexpr (NAN_OUT) {
    float m = vmax(__builtin_fabsf(v[0]), __builtin_fabsf(v[1]));
#pragma unroll
    for (int i = 2; i < 32; i += 2)
      m = vmax(m, vmax(__builtin_fabsf(v[i]), __builtin_fabsf(v[i + 1])));
    m = vmax(m, dpp_xor1(m));
    return vmax(m, dpp_xor2(m));
  } else {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(v[i]));
    m = __builtin_fmaxf(m, dpp_xor1(m));
    return __builtin_fmaxf(m, dpp_xor2(m));
  }
}

// A scale whose rounding to fp16 is relative (normal, not saturated) or 0:
// no quotient then exceeds (1 + 2^-11) q + 2^-20 < q + 1/2, q the largest
// code, and none needs a clamp.
__device__ __forceinline__ bool scale_exact(uint32_t s16) {
  return s16 == 0u || (s16 >= 0x0400u && s16 < 0x7bffu);
}

// Scale of the token and 1 / scale.  Where a token of the wave has a scale
// that is not exact in the above sense (or a NaN), all its values become
// their clamped quotients (a NaN the lowest) and inv becomes 1.
__device__ __forceinline__ uint32_t sym_scale(float v[32], float qm, float& inv) {
  uint32_t s = f16_sat(quad_amax<true>(v) / qm);
  const bool odd = __builtin_amdgcn_ballot_w64(!scale_exact(s)) != 0;
  if (odd) s = f16_sat(quad_amax<false>(v) / qm);
  const float sf = f16_to_f32((uint16_t)s);
  inv = sf != 0.0f ? 1.0f / sf : 0.0f;
  if (odd) {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = __builtin_amdgcn_fmed3f(v[i] * inv, -qm, qm);
    inv = 1.0f;
  }
  return s;
}

// Four codes as the bytes of a dword.
__device__ __forceinline__ uint32_t code_bytes(const uint32_t cb[4]) {
  return __builtin_amdgcn_perm(cb[1], cb[0], 0x0c0c0400u) |
         __builtin_amdgcn_perm(cb[3], cb[2], 0x04000c0cu);
}

// cb: kMagicBits + code
template <int B>
__device__ __forceinline__ void sym_key_chunk(const uint32_t cb[32], uint32_t* dst) {
  if constexpr (B <= 4) {
    ChunkAcc<B> acc;
    acc.init();
#pragma unroll
    for (int i = 0; i < 32; ++i) acc.add(i, cb[i]);
    acc.finish();
    store_chunk<B>(dst, acc.w);
  } else {
    uint32_t c[8], w[B];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = code_bytes(cb + 4 * i);
    pack_chunk<B>(c, w);
    store_chunk<B>(dst, w);
  }
}

// Two adjacent channels' chunks from their code bytes.
template <int B>
__device__ __forceinline__ void sym_value_chunks(const uint32_t c[2][8], uint32_t* dst) {
  uint32_t w[2 * B];
  pack_chunk<B>(c[0], w);
  pack_chunk<B>(c[1], w + B);
  store_chunk<2 * B>(dst, w);
}

// The block's value chunks (first: its first channel's number in the region)
// from the code bytes in LDS.
__device__ __forceinline__ void sym_values(const uint32_t* sm, int bits, uint32_t* region,
                                           size_t first, int lane) {
  __builtin_amdgcn_wave_barrier();
  // Lane -> the tokens of pass lane / 32 and channels 4 (lane % 32) .. + 3;
  // after the exchange of the wave's halves, all tokens of two channels.
  const int hf = lane >> 5, col = lane & 31;
  uint32_t tr[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    uint32_t r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int t = 4 * m + e;
      r[e] = sm[hf * kSymCodes + t * (kD / 4) + (((t >> 1) & 1) ? col ^ 4 : col)];
    }
    const uint32_t a01 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u);
    const uint32_t b01 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
    const uint32_t a23 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u);
    const uint32_t b23 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
    tr[0][m] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
    tr[1][m] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
    tr[2][m] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
    tr[3][m] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
  }
  uint32_t c[2][8];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const auto x = __builtin_amdgcn_permlane32_swap(tr[k][m], tr[2 + k][m], false, false);
      c[k][m] = x[0];
      c[k][4 + m] = x[1];
    }
  const size_t at = first + 4 * col + 2 * hf;
#define RQ_CASE(NB) \
  case NB: sym_value_chunks<NB>(c, region + at * NB); break;
  switch (bits) {
    RQ_CASE(2)
    RQ_CASE(3)
    RQ_CASE(4)
    RQ_CASE(5)
    RQ_CASE(6)
    RQ_CASE(7)
    RQ_CASE(8)
    default: break;
  }
#undef RQ_CASE
}

template <int ROT, int BF16>
__global__ void __launch_bounds__(kWave)
sym_quant_kernel(QuantLaunch a) {
  __shared__ __attribute__((aligned(16))) uint32_t sm[2 * kPass];
  const BlockId id = block_id(a);
  const int blk = id.blk, h = id.h, b = id.b, kind = id.kind;
  const int lane = threadIdx.x, tq = lane >> 2, q = lane & 3;
  const int nblk_cap = a.cap / kChunk, t0 = blk * kChunk;
  // The launch's window rows, a latency of memory: before the rest in a
  // decode step's wave (128 units, RTN 4.8 us with them behind, 4.6 so), else
  // behind (1000 tokens, RTN 5.1 us with them in front, 4.9 so).
  const bool ring_first = a.ring_fused == kRingAny && t0 < a.n_past;
  if (ring_first) copy_any(a, lane);
  stage_rows(a, b, h, kind, t0, lane, sm);
  const int bits = kernarg_byte(&a.tab.bits[0][0], 2 * h + kind);
  const int off = 1 << (bits - 1);
  const float qm = (float)(off - 1);
  // A code is rounded by one fp32 add of 2^23 + 2^(B-1) to the quotient:
  // half-to-even on the integer grid, and the even offset keeps the parity
  // of ties, so the low bits hold rint(quotient) + 2^(B-1).
  const float magic = 8388608.0f + (float)off;
  uint32_t* region = reinterpret_cast<uint32_t*>(a.codes + a.tab.code_off[h][kind]);
  const uint32_t neg = (ROT && (q == 1 || q == 2)) ? 0x80008000u : 0u;
  uint32_t scale[2];
  wait_rows<4>();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    float v[32];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u4 raw = *reinterpret_cast<const u4*>(
          &sm[slot(16 * p + tq, 4 * q + i)]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t ww = raw[e];
        if constexpr (ROT) {
          ww ^= neg;
          asm("" : "+v"(ww));    // (else negated per half)
        }
        v[8 * i + 2 * e] = widen_t<BF16>(ww & 0xffffu);
        v[8 * i + 2 * e + 1] = widen_t<BF16>(ww >> 16);
      }
    }
    if constexpr (ROT) rotate_quarter(v, q);
    float inv;
    scale[p] = sym_scale(v, qm, inv);
    uint32_t cb[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) cb[i] = __float_as_uint(v[i] * inv + magic);
    if (p == 0) wait_rows<0>();     // (here, not after the codes' stores)
    if (kind == 0) {
      // keys: this lane's chunk packed from registers
      const size_t at = ((size_t)b * a.cap + t0 + 16 * p + tq) * 4 + q;
#define RQ_CASE(NB) \
  case NB: sym_key_chunk<NB>(cb, region + at * NB); break;
      switch (bits) {
        RQ_CASE(2)
        RQ_CASE(3)
        RQ_CASE(4)
        RQ_CASE(5)
        RQ_CASE(6)
        RQ_CASE(7)
        RQ_CASE(8)
        default: break;
      }
#undef RQ_CASE
    } else {
      // values: code bytes staged as [token][channel] for the transpose, in
      // place of the rows read above (a wave's LDS operations keep their
      // order); the
      // two 16-byte stores of a lane are exchanged for two tokens in four, so
      // that the 16 lanes of a store's turn take all banks
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        u4 d;
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = code_bytes(cb + 16 * i + 4 * e);
        const int at = 8 * q + 4 * (i ^ ((tq >> 1) & 1));
        *reinterpret_cast<u4*>(&sm[p * kSymCodes + tq * (kD / 4) + at]) = d;
      }
    }
  }
  if (q == 0) {
    // tokens t and t + 16: a pair of the metadata's order
    uint32_t* m = reinterpret_cast<uint32_t*>(
        a.meta + meta_unit_offset(a.family, h, kind, b, a.B, nblk_cap) +
        (size_t)blk * kMetaBlockTok);
    __builtin_nontemporal_store(scale[0] | (scale[1] << 16), gptr(m) + tq);
  }
  if (kind == 1) sym_values(sm, bits, region, ((size_t)b * nblk_cap + blk) * kD, lane);
  if (!ring_first) copy_ring(a, id, lane);
}

__global__ void __launch_bounds__(kWave)
ring_kernel(RingLaunch a) {
  const int t = a.t_lo + blockIdx.x;
  const int h = blockIdx.y;
  const int b = blockIdx.z >> 1, kind = blockIdx.z & 1;
  const uint16_t* base = kind ? a.v : a.k;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(
      base + ((size_t)(b * a.H + h) * a.n_new + (t - a.n_past)) * kD);
  const int cap = a.R + kChunk;
  uint32_t* dst = reinterpret_cast<uint32_t*>(
      a.resid + ((((size_t)b * a.H + h) * 2 + kind) * cap + (t % cap)) * kD);
  dst[threadIdx.x] = src[threadIdx.x];
}

// A launch that reads more than this marks its loads non-temporal: they pass
// by the caches, which then keep what the rest of the program uses.  Below it
// the input, just written by the projections, is likely still in the 256 MiB
// of last-level cache and plain loads find it there.  (RTN 4 bits, 8 kv-heads,
// plain / non-temporal: 32 MiB 8.76 / 9.15 us, 64 MiB 15.5 / 16.6, 128 MiB
// 31.7 / 30.5, 256 MiB 63.0 / 60.9, 512 MiB 123.3 / 119.0; right after the
// matrix products that write the input: RTN 4 bits 64 MiB 20.5 / 19.8, 96 MiB
// 26.7 / 27.1, 192 MiB 47.8 / 42.8, KIVI 3 bits 27.1 / 28.1 and 52.5 / 46.9.
// Only an input of 96 to 256 MiB that lies in that cache already, such as one
// quantized again and again, is read faster by plain loads: 192 MiB, RTN 3
// bits 36.6 / 45.2.)
constexpr size_t kStreamBytes = (size_t)96 << 20;

// Workgroups in order of the blocks of a unit, then the kv-heads and kinds of
// a batch entry (the inputs' order), or, for units of at least 6144 tokens,
// the batch entries of a head and kind (the codes' order, and one width at a
// time): KIVI 2.5 bits, 8 kv-heads, by batch / by head, us: 16 x 2048 tokens
// 31.2 / 32.9, 64 x 2048 114.1 / 122.5, 16 x 4096 58.8 / 58.5, 32 x 4096
// 113.3 / 114.0, 11 x 8192 80.7 / 78.8, 16 x 8192 115.5 / 107.9, 16 x 16384
// 225.9 / 212.7.  The other kernels: 64 x 2048 RTN 4 bits 110 / 128, QuaRot
// 116 / 128, KIVI_RTN 114 / 124; 16 x 8192 RTN 4 bits 127 / 114, 3 bits 107 /
// 108, QuaRot 4 bits 130 / 114, 2..6 bits 119 / 121, KIVI 4 bits 133 / 116, 2..6
// bits 124 / 123, KIVI_RTN 112 / 116 (by batch, power-of-two strides of 4-bit
// codes collide); 8 x 16384 in that order 123 / 105, 106 / 101, 135 / 108, 119 /
// 115, 131 / 110, 123 / 118, 111 / 106.
dim3 set_grid(QuantLaunch& q) {
  q.stream = (size_t)q.nblk * q.H * q.B * q.kind_n * (kChunk * kD * 2) > kStreamBytes;
  q.by_batch = q.nblk < 192 && q.B <= 65535;      // (the grid's limit along z)
  return q.by_batch ? dim3(q.nblk, q.H * q.kind_n, q.B) : dim3(q.nblk * q.B, q.H * q.kind_n);
}

// KIVI blocks of kinds q.kind_lo .. + q.kind_n - 1
hipError_t launch_kivi(QuantLaunch q, hipStream_t s) {
  int maxb = 1;
  for (int h = 0; h < q.H; ++h)
    for (int k = q.kind_lo; k < q.kind_lo + q.kind_n; ++k)
      maxb = q.tab.bits[h][k] > maxb ? q.tab.bits[h][k] : maxb;
  const dim3 grid = set_grid(q), block(kWave);
  if (maxb <= 4) {
    if (q.is_bf16)
      hipLaunchKernelGGL((kivi_quant_kernel<1, 4>), grid, block, 0, s, q);
    else
      hipLaunchKernelGGL((kivi_quant_kernel<0, 4>), grid, block, 0, s, q);
  } else {
    if (q.is_bf16)
      hipLaunchKernelGGL((kivi_quant_kernel<1, 8>), grid, block, 0, s, q);
    else
      hipLaunchKernelGGL((kivi_quant_kernel<0, 8>), grid, block, 0, s, q);
  }
  return hipGetLastError();
}

// per-token symmetric blocks (QuaRot with the rotation, RTN without) of
// kinds q.kind_lo .. + q.kind_n - 1
hipError_t launch_sym(QuantLaunch q, bool rot, hipStream_t s) {
  const dim3 grid = set_grid(q);
  // bit-widths of the symmetric quantizers are 2..8 (checked on the host)
  if (rot && q.is_bf16)
    hipLaunchKernelGGL((sym_quant_kernel<1, 1>), grid, dim3(kWave), 0, s, q);
  else if (rot)
    hipLaunchKernelGGL((sym_quant_kernel<1, 0>), grid, dim3(kWave), 0, s, q);
  else if (q.is_bf16)
    hipLaunchKernelGGL((sym_quant_kernel<0, 1>), grid, dim3(kWave), 0, s, q);
  else
    hipLaunchKernelGGL((sym_quant_kernel<0, 0>), grid, dim3(kWave), 0, s, q);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_quantize(const QuantLaunch& a, hipStream_t s) {
  if (a.nblk <= 0) return hipSuccess;
  QuantLaunch q = a;
  q.kind_lo = 0;
  q.kind_n = 2;
  if (a.family == RQ_TURBO) return launch_quantize_turbo(q, s);
  if (a.family == RQ_KIVI) return launch_kivi(q, s);
  if (a.family == RQ_KIVI_RTN) {
    // keys by KIVI, values by RTN
    q.kind_n = 1;
    hipError_t e = launch_kivi(q, s);
    if (e != hipSuccess) return e;
    q.kind_lo = 1;
    if (q.ring_fused == kRingAny) q.ring_fused = 0;   // copied by the keys' launch
    return launch_sym(q, false, s);
  }
  return launch_sym(q, a.family == RQ_QUAROT, s);
}

hipError_t launch_ring(const RingLaunch& a, hipStream_t s) {
  if (a.t_hi <= a.t_lo) return hipSuccess;
  dim3 grid(a.t_hi - a.t_lo, a.H, a.B * 2);
  hipLaunchKernelGGL(ring_kernel, grid, dim3(kWave), 0, s, a);
  return hipGetLastError();
}

}  // namespace rq
