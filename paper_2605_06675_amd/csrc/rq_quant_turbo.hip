// TurboQuant-style quantize + pack (Sec. 2; Sec. 3.1 and Table 6 for the
// codebook): per token, y = R x with the (layer, kv-head) rotation R, the
// norm n = |x| (fp16), and per coordinate the code of t = y sqrt(128) / n
// among the b-bit Lloyd-Max thresholds of N(0,1).
//
// A workgroup serves one kv-head: R sits in LDS and its four waves loop over
// that head's blocks (block, batch entry, K|V).  A block's 16-bit rows are
// loaded straight into matrix-core operands:
//   keys   D[coord][token] = R . X^T   (the chunk of a token is 32 coords)
//   values D[token][coord] = X . R^T   (the chunk of a coord is 32 tokens)
// on v_mfma_f32_16x16x32 (bf16 inputs; fp16 inputs with R converted to
// fp16, exact for the entries of magnitude 2^-17 and above, about one entry
// of a Haar matrix rounding to the fp16 subnormal grid, by at most 2^-25).
// Norms come from the same registers (exact; see norm_of).  Codes count the
// positive thresholds below |t| (the codebook is symmetric, with the middle
// threshold at 0).  Every lane holds quarters of chunks; permlane swaps turn
// four lanes' quarters into whole chunks, which each lane packs and stores.
//
// What bounds it: vector instructions (about 770 a block of 4096 elements,
// 1380 before the tables, the fp32 norms and the transposes in registers)
// and the 64 matrix instructions, 83 and 27 us of the launch at 2.4 GHz,
// which overlap only in part; memory alone takes 116 us.  Llama-3-70B layer
// (4 x 8 units of 32768 tokens, 2..4 bits at 3.0): 207 us before, 149 us
// now; at 5.25 bits on average (a count of 2 P comparisons before) 260 us
// and 93 us for 4 x 8 x 15584 tokens.  Four workgroups a CU without a
// second register buffer (112 registers) beat three with one (149 and 157
// us): the other waves' work covers the loads.
#include "rq_device.h"
#include "rq_internal.h"
#include "rq_ring.h"

namespace rq {

namespace {

constexpr int kWave = 64;
constexpr int kTWaves = 4;       // waves per workgroup
constexpr int kTOcc = 4;         // workgroups per CU
constexpr float kSqrtD = 11.313708498984761f;   // fp32 nearest to sqrt(128)

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

template <int BF16>
__device__ __forceinline__ f4 mma(u4 a, u4 b, f4 c) {
  if constexpr (BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a),
                                                   __builtin_bit_cast(bf8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a),
                                                  __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

template <int BF16>
__device__ __forceinline__ float wid(uint32_t w16) {
  if (BF16) return __uint_as_float(w16 << 16);
  return (float)__builtin_bit_cast(_Float16, (uint16_t)w16);
}

// bf16 -> fp16 bit pattern: exact for |r| >= 2^-17 (the 8 significant bits
// of a bf16 value fit the fp16 grid there); smaller entries round to the
// fp16 subnormal grid (spacing 2^-24)
__device__ __forceinline__ uint32_t bf16_to_f16(uint32_t b) {
  return __builtin_bit_cast(uint16_t, (_Float16)__uint_as_float(b << 16));
}

struct TBlock {
  int blk, b, kind;
};

__device__ __forceinline__ TBlock turbo_block(const QuantLaunch& a, int it) {
  TBlock id;
  id.blk = a.blk0 + it % a.nblk;
  const int z = it / a.nblk;
  id.b = z >> 1;
  id.kind = z & 1;
  return id;
}

__device__ __forceinline__ const uint16_t* row_src(const QuantLaunch& a, int b, int h,
                                                   int kind, int t) {
  if (t >= a.n_past) {
    const uint16_t* base = kind ? a.v : a.k;
    return base + ((size_t)(b * a.H + h) * a.n_new + (t - a.n_past)) * kD;
  }
  const int cap = a.R + kChunk;
  return a.resid + ((((size_t)b * a.H + h) * 2 + kind) * cap + (t % cap)) * kD;
}

// Operand registers of a block: x[4 tt + ks] holds, in lane l, 16-bit
// channels 32 ks + 8 (l / 16) .. + 7 of token 16 tt + l % 16.
__device__ __forceinline__ void load_x(const QuantLaunch& a, int h, const TBlock& id,
                                       u4 x[8], int lane) {
  const int t0 = id.blk * kChunk;
  const int g = lane >> 4, j = lane & 15;
  if (t0 >= a.n_past) {
    const RQ_GLOBAL u4* src = gptr(reinterpret_cast<const u4*>(
        (id.kind ? a.v : a.k) +
        ((size_t)(id.b * a.H + h) * a.n_new + (t0 - a.n_past)) * kD));
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) x[4 * tt + ks] = src[(16 * tt + j) * 16 + 4 * ks + g];
  } else {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const RQ_GLOBAL u4* row = gptr(reinterpret_cast<const u4*>(
          row_src(a, id.b, h, id.kind, t0 + 16 * tt + j)));
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) x[4 * tt + ks] = row[4 * ks + g];
    }
  }
}

// R in LDS: rows of 256 bytes whose 16-byte pieces are stored at place
// piece ^ (row mod 16), so that the lanes of an operand read (16 rows, four
// pieces each) spread over all banks (rows padded to 272 bytes, in
// comparison, cost 4 cycles of conflicts a read of 8).
__device__ __forceinline__ int r_place(int row, int piece) {
  return row * kD + 8 * (piece ^ (row & 15));
}
// R operand of coordinate tile ct, k-step ks: lane l holds R[16 ct + l % 16]
// [32 ks + 8 (l / 16) .. + 7] (the A operand of R . X^T and the B operand of
// X . R^T have the same lane layout).  at[ks] = r_place(l % 16, 4 ks + l / 16).
__device__ __forceinline__ u4 r_op(const uint16_t* Rs, const int (&at)[4], int ct, int ks) {
  return *reinterpret_cast<const u4*>(Rs + at[ks] + 16 * ct * kD);
}

// ---------------------------------------------------------------- norms
// n16[tt] = fp16 of fp32(sqrt(sum of squares)) of token 16 tt + lane % 16,
// the sum and the root in fp64.
template <int BF16>
__device__ __forceinline__ uint32_t norm_exact(const u4* x) {
  double s = 0.0;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const u4 w = x[ks];
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double lo = (double)wid<BF16>(ww[e] & 0xffffu);
      const double hi = (double)wid<BF16>(ww[e] >> 16);
      s = __builtin_fma(lo, lo, s);
      s = __builtin_fma(hi, hi, s);
    }
  }
  s += __shfl_xor(s, 16, kWave);
  s += __shfl_xor(s, 32, kWave);
  return f16_sat((float)__builtin_sqrt(s));
}

// The same from an fp32 sum wherever that settles the fp16 result.  The 32
// squares of a lane are exact in fp32 and are added in two chains of 16,
// then over the four lanes of the token: at most 19 roundings on any path,
// of 2^-23 at the most each whatever way v_dot2 rounds, all terms >= 0.  So
// the sum is within 2^-18.7 of the exact one and its root within 2^-19.7;
// v_sqrt_f32 and the scaling below add less than 2^-22 more.  kNormEps
// bounds all of it: where n (1 - eps) and n (1 + eps) round to the same fp16
// value, so does the exact root (rounding is monotone, and fp32 rounding
// before fp16 stays inside the interval).  Sums that underflow belong to
// norms far below fp16's least subnormal, sums that overflow to norms that
// saturate: both settle at their true value.  About one token in 150 does
// not settle; its sixteen tokens go through fp64.  Half an instruction an
// element (fp16: one) in place of about 7.
constexpr float kNormEps = 1.9073486328125e-6f;   // 2^-19

template <int BF16>
__device__ __forceinline__ uint32_t norm_of(const u4* x) {
  float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const u4 w = x[ks];
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (BF16) {
        typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
        const bf2 v = __builtin_bit_cast(bf2, ww[e]);
        float& s = (e & 1) ? s1 : s0;
        s = __builtin_amdgcn_fdot2_f32_bf16(v, v, s, false);
      } else {
        const float lo = wid<BF16>(ww[e] & 0xffffu), hi = wid<BF16>(ww[e] >> 16);
        s0 = __builtin_fmaf(lo, lo, s0);
        s1 = __builtin_fmaf(hi, hi, s1);
      }
    }
  }
  float s = s0 + s1;
  s += __shfl_xor(s, 16, kWave);
  s += __shfl_xor(s, 32, kWave);
  const float n = __builtin_amdgcn_sqrtf(s);
  const uint32_t lo = f16_sat(n * (1.0f - kNormEps)), hi = f16_sat(n * (1.0f + kNormEps));
  if (__builtin_amdgcn_ballot_w64(lo != hi || !(s >= 0.0f))) return norm_exact<BF16>(x);
  return lo;
}

// ---------------------------------------------------------------- codes
// The code of t is the number of thresholds below t.  The L - 1 thresholds
// are -th reversed, 0, th (th: the P = L/2 - 1 positive ones, ascending);
// with cnt = #{j : th[j] < |t|} the code is L/2 + cnt for t > 0, else
// L/2 - 1 - cnt.  A lane's eight codes of a chunk (4g + i and 16 + 4g + i,
// i = 0..3: quarter g = lane / 16) are gathered as fields [t < 0][cnt] and
// turned into codes together (codes_of_fields).  The sign is t's sign bit,
// and t = 0 (a zero coordinate, a token of norm zero) belongs to the
// negative side: t is formed by a fused multiply-add of -2^-149, fp32's
// least subnormal, which leaves every other rounded product as it is (but for
// one halfway between two fp32 values, which may round the other way).
//
// Widths 1..3: the bits of a field are compared one by one (bisection over
// th) and shifted into the quarter's dword, one add with carry per bit, so
// that the fields land where the chunk wants them: adjacent for three bits
// (stream bits 24g ..), else the four codes of each half in their half-word.
// Widths 4..8: cnt from a table in LDS.  The cell of |t|, floor(|t| 2^(b-2)),
// holds at most one threshold (the least gap of the codebook is 1.03 ..
// 1.08 cells) and the count of those in lower cells; t arrives multiplied by
// 2^(b-2), which is exact.  Eight instructions and one LDS read a code at
// every width, where bisection takes 13 at four bits and a count over all
// thresholds 2 P (30 .. 254) above.
__host__ __device__ constexpr int turbo_cells(int b) {
  return b == 4 ? 16 : b == 5 ? 32 : b == 6 ? 64 : b == 7 ? 136 : 288;
}
constexpr int kMaxCells = 288;
struct Cell {
  float th;        // the cell's threshold times 2^(b-2), or +inf
  uint32_t below;  // positive thresholds in lower cells
};

__device__ __forceinline__ uint32_t cell_of(float ts, int cells) {
  // (clamped as a float: a token of saturated norm reaches values whose
  // conversion is not defined; a NaN takes cell 0)
  return (uint32_t)__builtin_amdgcn_fmed3f(__builtin_fabsf(ts), 0.0f, (float)(cells - 1));
}

// Tables of the head's K (kind 0) and V widths; whole workgroup.
__device__ __forceinline__ void fill_cells(const QuantLaunch& a, int h, Cell (*tab)[kMaxCells]) {
  static_assert(kTWaves * kWave == 256, "128 threads per table");
  const int kind = threadIdx.x >> 7, k = threadIdx.x & 127;
  const int b = kernarg_byte(&a.tab.bits[0][0], 2 * h + kind);
  if (b < 4) return;
  const int P = (1 << (b - 1)) - 1, cells = turbo_cells(b);
  if (k >= P) return;
  const RQ_GLOBAL float* tp = gptr(a.cb + (b - 1) * 512 + (1 << (b - 1)));
  const float scale = (float)(1 << (b - 2));
  const float th = tp[k] * scale;
  const int c = (int)cell_of(th, cells);
  const int next = k + 1 < P ? (int)cell_of(tp[k + 1] * scale, cells) : cells;
  if (k == 0)
    for (int i = 0; i < c; ++i) tab[kind][i] = Cell{INFINITY, 0u};
  tab[kind][c] = Cell{th, (uint32_t)k};
  for (int i = c + 1; i < next; ++i) tab[kind][i] = Cell{INFINITY, (uint32_t)k + 1u};
}

template <int B> struct Quarter {
  // widths 5..8: one dword of code bytes per half; else one dword in all
  static constexpr int n = B >= 5 ? 2 : 1;
  uint32_t w[n];
};

// Two more fields at the low end of acc (widths 1..3): that of ta, then that
// of tb.  Written out, since the compiler turns the add with carry into a
// select, a shift and an or (12 instructions a three-bit code in place of 7);
// a mask is read at the earliest two instructions after the comparison that
// writes it, as the hardware wants.
#define RQ_CMP(S, T, TH) "v_cmp_gt_f32_e64 %" S ", |%" T "|, %" TH "\n\t"
#define RQ_SEL(D, LO, HI, S) "v_cndmask_b32_e64 %" D ", %" LO ", %" HI ", %" S "\n\t"
#define RQ_SIGN(T) "v_alignbit_b32 %[acc], %[acc], %" T ", 31\n\t"
#define RQ_PUSH(S) "v_addc_co_u32_e64 %[acc], vcc, %[acc], %[acc], %" S "\n\t"
template <int B>
__device__ __forceinline__ void push_fields(uint32_t& acc, float ta, float tb, const float* th) {
  uint64_t ma, mb, na, nb;
  float xa, xb;
  if constexpr (B == 1) {
    acc = __builtin_amdgcn_alignbit(acc, __float_as_uint(ta), 31);
    acc = __builtin_amdgcn_alignbit(acc, __float_as_uint(tb), 31);
  } else if constexpr (B == 2) {
    asm(RQ_CMP("[ma]", "[ta]", "[t0]") RQ_CMP("[mb]", "[tb]", "[t0]")
        RQ_SIGN("[ta]") RQ_PUSH("[ma]") RQ_SIGN("[tb]") RQ_PUSH("[mb]")
        : [acc] "+v"(acc), [ma] "=&s"(ma), [mb] "=&s"(mb)
        : [ta] "v"(ta), [tb] "v"(tb), [t0] "v"(th[0])
        : "vcc");
  } else {
    asm(RQ_CMP("[ma]", "[ta]", "[t1]") RQ_CMP("[mb]", "[tb]", "[t1]")
        RQ_SIGN("[ta]")
        RQ_SEL("[xa]", "[t0]", "[t2]", "[ma]") RQ_SEL("[xb]", "[t0]", "[t2]", "[mb]")
        RQ_CMP("[na]", "[ta]", "[xa]") RQ_CMP("[nb]", "[tb]", "[xb]")
        RQ_PUSH("[ma]") RQ_PUSH("[na]") RQ_SIGN("[tb]") RQ_PUSH("[mb]") RQ_PUSH("[nb]")
        : [acc] "+v"(acc), [ma] "=&s"(ma), [mb] "=&s"(mb), [na] "=&s"(na), [nb] "=&s"(nb),
          [xa] "=&v"(xa), [xb] "=&v"(xb)
        : [ta] "v"(ta), [tb] "v"(tb), [t0] "v"(th[0]), [t1] "v"(th[1]), [t2] "v"(th[2])
        : "vcc");
  }
}
#undef RQ_CMP
#undef RQ_SEL
#undef RQ_SIGN
#undef RQ_PUSH

// Sign bits of a quarter's fields (widths 5..8: of one half's code bytes).
__host__ __device__ constexpr uint32_t field_signs(int b) {
  return b == 1 ? 0x000f000fu : b == 2 ? 0x00aa00aau : b == 3 ? 0x00924924u
       : b == 4 ? 0x88888888u : 0x01010101u << (b - 1);
}
// Fields [t < 0][cnt] to codes: L/2 + cnt, or L/2 - 1 - cnt where negative
// (m - (m >> (b - 1)), m the set sign bits, is the mask of their cnt bits).
template <int B>
__device__ __forceinline__ uint32_t codes_of_fields(uint32_t f) {
  constexpr uint32_t signs = field_signs(B);
  const uint32_t m = f & signs;
  return f ^ signs ^ (B > 1 ? m - (m >> (B - 1)) : 0u);
}

__device__ __forceinline__ float t_of(float y, float f) {
  return __builtin_fmaf(y, f, -1.40129846432481707e-45f);
}

// The quarter of codes y0[i] f0[i] (codes 4g + i) and y1[i] f1[i]
// (16 + 4g + i).
template <int B>
__device__ __forceinline__ Quarter<B> quarter_codes(f4 y0, f4 y1, const float* f0,
                                                    const float* f1, const float* th,
                                                    const Cell* tab) {
  Quarter<B> q;
  if constexpr (B >= 4) {
    // the fields of a half as code bytes, or (four bits) as a half-word
    constexpr int stride = B == 4 ? 4 : 8;
    uint32_t acc = 0;
#pragma unroll
    for (int c = 1; c >= 0; --c) {
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        const float t = c ? t_of(y1[i], f1[i]) : t_of(y0[i], f0[i]);
        const Cell e = tab[cell_of(t, turbo_cells(B))];
        const uint32_t cnt = e.below + (e.th < __builtin_fabsf(t) ? 1u : 0u);
        acc = __builtin_amdgcn_alignbit(acc << (stride - B), __float_as_uint(t), 31);
        acc = (acc << (B - 1)) | cnt;
      }
      if constexpr (B >= 5) q.w[c] = codes_of_fields<B>(acc);
    }
    if constexpr (B == 4) q.w[0] = codes_of_fields<B>(acc);
  } else {
    uint32_t acc = 0;
    push_fields<B>(acc, t_of(y1[3], f1[3]), t_of(y1[2], f1[2]), th);
    push_fields<B>(acc, t_of(y1[1], f1[1]), t_of(y1[0], f1[0]), th);
    if constexpr (B < 3) acc <<= 16 - 4 * B;
    push_fields<B>(acc, t_of(y0[3], f0[3]), t_of(y0[2], f0[2]), th);
    push_fields<B>(acc, t_of(y0[1], f0[1]), t_of(y0[0], f0[0]), th);
    q.w[0] = codes_of_fields<B>(acc);
  }
  return q;
}

// Transpose of four registers over the four 16-lane rows of the wave:
// afterwards register r of row g holds what register g of row r held.
__device__ __forceinline__ void transpose_rows(uint32_t& a0, uint32_t& a1, uint32_t& a2,
                                               uint32_t& a3) {
  const auto p = __builtin_amdgcn_permlane32_swap(a0, a2, false, false);
  const auto r = __builtin_amdgcn_permlane32_swap(a1, a3, false, false);
  const auto s = __builtin_amdgcn_permlane16_swap(p[0], r[0], false, false);
  const auto t = __builtin_amdgcn_permlane16_swap(p[1], r[1], false, false);
  a0 = s[0];
  a1 = s[1];
  a2 = t[0];
  a3 = t[1];
}

// Four chunks' quarters (q[c]: this lane's quarter g of chunk c) to one
// whole chunk per lane (chunk g), packed and stored at dst (B words).
template <int B>
__device__ __forceinline__ void store_chunks(Quarter<B> (&q)[4], uint32_t* dst) {
#pragma unroll
  for (int k = 0; k < Quarter<B>::n; ++k)
    transpose_rows(q[0].w[k], q[1].w[k], q[2].w[k], q[3].w[k]);
  uint32_t w[B];
  if constexpr (B == 1) {
    w[0] = q[0].w[0] | (q[1].w[0] << 4) | (q[2].w[0] << 8) | (q[3].w[0] << 12);
  } else if constexpr (B == 2) {
    w[0] = q[0].w[0] | (q[1].w[0] << 8);
    w[1] = q[2].w[0] | (q[3].w[0] << 8);
  } else if constexpr (B == 3) {
    // words 0..2 = stream bits 0..31, 32..63, 64..95
    w[0] = q[0].w[0] | (q[1].w[0] << 24);
    w[1] = __builtin_amdgcn_alignbit(q[2].w[0], q[1].w[0] << 8, 16);
    w[2] = __builtin_amdgcn_alignbit(q[3].w[0], q[2].w[0] << 8, 24);
  } else if constexpr (B == 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = q[i].w[0];
  } else {
    const uint32_t c[8] = {q[0].w[0], q[1].w[0], q[2].w[0], q[3].w[0],
                           q[0].w[1], q[1].w[1], q[2].w[1], q[3].w[1]};
    pack_chunk<B>(c, w);
  }
  RQ_GLOBAL uint32_t* d = gptr(dst);
#pragma unroll
  for (int i = 0; i < B; ++i) __builtin_nontemporal_store(w[i], d + i);
}

template <int BF16, int B>
__device__ __forceinline__ void turbo_block_codes(const QuantLaunch& a, const uint16_t* Rs,
                                                  const Cell* tab, int h, const TBlock& id,
                                                  const u4 x[8], int lane) {
  constexpr int L = 1 << B, P = L / 2 - 1;
  // what follows from the lane is computed per block: hoisted out of the
  // block loop, the store offsets of eight widths would hold registers
  asm volatile("" : "+v"(lane));
  const int g = lane >> 4, j = lane & 15;
  const int t0 = id.blk * kChunk;
  int at[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) at[ks] = r_place(j, 4 * ks + g);
  float th[B <= 3 && P > 0 ? P : 1];
  if constexpr (B <= 3) {
    const RQ_GLOBAL float* tp = gptr(a.cb + (B - 1) * 512 + L / 2);
#pragma unroll
    for (int k = 0; k < P; ++k) th[k] = tp[k];
  }
  // tokens 16 tt + j: norms, and the factors y -> t (times 2^(B-2), the cell
  // scale, for the wider codes)
  float f[2];
  uint32_t n16[2];
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    n16[tt] = norm_of<BF16>(x + 4 * tt);
    const float nf = f16_to_f32((uint16_t)n16[tt]);
    f[tt] = nf != 0.0f ? kSqrtD / nf : 0.0f;
    if constexpr (B >= 4) f[tt] *= (float)(1 << (B - 2));
  }
  // metadata: token 16 tt + j at pair position 2 j + tt
  const int nblk_cap = a.cap / kChunk;
  if (g == 0) {
    RQ_GLOBAL uint32_t* m = gptr(reinterpret_cast<uint32_t*>(
        a.meta + ((((size_t)h * 2 + id.kind) * a.B + id.b) * nblk_cap + id.blk) *
                     kMetaBlockTok));
    m[j] = n16[0] | (n16[1] << 16);
  }
  uint32_t* region = reinterpret_cast<uint32_t*>(a.codes + a.tab.code_off[h][id.kind]);
  if (id.kind == 0) {
    // keys: chunk q of token 16 tt + j = coordinate tiles 2q, 2q + 1; lane:
    // token 16 tt + j, coords 32q + 16c + 4g + i -> code 16c + 4g + i
    uint32_t* base = region + ((size_t)id.b * a.cap + t0) * 4 * B;
    const float f0[4] = {f[0], f[0], f[0], f[0]}, f1[4] = {f[1], f[1], f[1], f[1]};
    Quarter<B> qt[2][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f4 d[2][2];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) d[c][tt] = (f4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const u4 r0 = r_op(Rs, at, 2 * q, ks), r1 = r_op(Rs, at, 2 * q + 1, ks);
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
          d[0][tt] = mma<BF16>(r0, x[4 * tt + ks], d[0][tt]);
          d[1][tt] = mma<BF16>(r1, x[4 * tt + ks], d[1][tt]);
        }
      }
      qt[0][q] = quarter_codes<B>(d[0][0], d[1][0], f0, f0, th, tab);
      qt[1][q] = quarter_codes<B>(d[0][1], d[1][1], f1, f1, th, tab);
      // one chunk's tiles at a time: the unrolled steps otherwise overlap
      // beyond the registers there are
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
      store_chunks<B>(qt[tt], base + ((16 * tt + j) * 4 + g) * B);
  } else {
    // values: chunk of coord 16 ct + j = its 32 tokens; lane: tokens
    // 16 tt + 4g + i -> code 16 tt + 4g + i
    uint32_t* base = region + ((size_t)id.b * nblk_cap + id.blk) * kD * B;
    float fr[2][4];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) fr[tt][i] = __shfl(f[tt], 4 * g + i, kWave);
#pragma unroll
    for (int c4 = 0; c4 < 2; ++c4) {
      Quarter<B> qt[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        f4 d[2] = {(f4){0.0f, 0.0f, 0.0f, 0.0f}, (f4){0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const u4 r = r_op(Rs, at, 4 * c4 + c, ks);
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) d[tt] = mma<BF16>(x[4 * tt + ks], r, d[tt]);
        }
        qt[c] = quarter_codes<B>(d[0], d[1], fr[0], fr[1], th, tab);
        __builtin_amdgcn_sched_barrier(0);
      }
      store_chunks<B>(qt, base + (16 * (4 * c4 + g) + j) * B);
    }
  }
}

template <int BF16>
__device__ __forceinline__ void turbo_dispatch(const QuantLaunch& a, const uint16_t* Rs,
                                               const Cell (*tab)[kMaxCells], int h,
                                               const TBlock& id, const u4 x[8], int lane) {
  const Cell* cells = tab[id.kind];
  switch (kernarg_byte(&a.tab.bits[0][0], 2 * h + id.kind)) {
    case 1: turbo_block_codes<BF16, 1>(a, Rs, cells, h, id, x, lane); break;
    case 2: turbo_block_codes<BF16, 2>(a, Rs, cells, h, id, x, lane); break;
    case 3: turbo_block_codes<BF16, 3>(a, Rs, cells, h, id, x, lane); break;
    case 4: turbo_block_codes<BF16, 4>(a, Rs, cells, h, id, x, lane); break;
    case 5: turbo_block_codes<BF16, 5>(a, Rs, cells, h, id, x, lane); break;
    case 6: turbo_block_codes<BF16, 6>(a, Rs, cells, h, id, x, lane); break;
    case 7: turbo_block_codes<BF16, 7>(a, Rs, cells, h, id, x, lane); break;
    case 8: turbo_block_codes<BF16, 8>(a, Rs, cells, h, id, x, lane); break;
    default: break;
  }
}

// grid (workgroups per head, kv-heads)
template <int BF16>
__global__ void __launch_bounds__(kTWaves * kWave, kTOcc)
turbo_quant_kernel(QuantLaunch a) {
  __shared__ uint16_t Rs[kD * kD];
  __shared__ Cell cells[2][kMaxCells];
  const int h = blockIdx.y;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  {
    // R of this head, 16-byte pieces (row i / 16, piece i % 16)
    const RQ_GLOBAL u4* src = gptr(reinterpret_cast<const u4*>(a.rot + (size_t)h * kD * kD));
    for (int i = threadIdx.x; i < kD * 16; i += kTWaves * kWave) {
      u4 v = src[i];
      if (!BF16) {
        v.x = bf16_to_f16(v.x & 0xffffu) | (bf16_to_f16(v.x >> 16) << 16);
        v.y = bf16_to_f16(v.y & 0xffffu) | (bf16_to_f16(v.y >> 16) << 16);
        v.z = bf16_to_f16(v.z & 0xffffu) | (bf16_to_f16(v.z >> 16) << 16);
        v.w = bf16_to_f16(v.w & 0xffffu) | (bf16_to_f16(v.w >> 16) << 16);
      }
      *reinterpret_cast<u4*>(&Rs[r_place(i >> 4, i & 15)]) = v;
    }
  }
  fill_cells(a, h, cells);
  __syncthreads();
  const int per_head = a.nblk * a.B * 2;
  const int stride = gridDim.x * kTWaves;
  int it = blockIdx.x * kTWaves + wave;
  for (; it < per_head; it += stride) {
    const TBlock id = turbo_block(a, it);
    u4 x[8];
    load_x(a, h, id, x, lane);
    turbo_dispatch<BF16>(a, Rs, cells, h, id, x, lane);
  }
  // the window rows of the append, after the blocks (fewer live registers)
  if (a.ring_fused)
    copy_window(a.ring, (blockIdx.y * gridDim.x + blockIdx.x) * kTWaves + wave,
                gridDim.x * gridDim.y * kTWaves, lane);
}

}  // namespace

hipError_t launch_quantize_turbo(const QuantLaunch& a, hipStream_t s) {
  if (a.nblk <= 0) return hipSuccess;
  const long per_head = (long)a.nblk * a.B * 2;
  long per = ((long)(a.n_cu > 0 ? a.n_cu : 256) * kTOcc + a.H - 1) / a.H;
  const long need = (per_head + kTWaves - 1) / kTWaves;
  if (per > need) per = need;
  if (per < 1) per = 1;
  dim3 grid((unsigned)per, a.H), block(kTWaves * kWave);
  if (a.is_bf16)
    hipLaunchKernelGGL(turbo_quant_kernel<1>, grid, block, 0, s, a);
  else
    hipLaunchKernelGGL(turbo_quant_kernel<0>, grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace rq
