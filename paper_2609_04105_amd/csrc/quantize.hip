// MXFP4 and MXFP8 input quantizers.
//
// Quantizer (eq. mx-scale): per block of 32 values with absolute maximum a,
// the E8M0 amplitude is 2^floor(log2 a) or 2^ceil(log2 a), whichever has the
// smaller squared reconstruction error (ties keep the ceiling).  With
// r = 6|v| / 2^e_ceil, ceiling codes qc = E2M1(r) and floor codes qf = E2M1(2r),
// the floor wins iff sum (2 qc - qf)(4 r - qf - 2 qc) < 0; every term of that
// sum is exact in fp64 for fp32/bf16 inputs, so the choice is exact.
// Both input types take 32-bit paths with the hardware E2M1 converter (exact
// too, see mxfp4_block_bf16 and mxfp4_block_f32).  One thread owns one block.
//
// What bounds it: memory.  Each value is read once (2 or 4 bytes) and leaves as
// 17/32 byte (MXFP8: 33/32).  Q, K and V of B2 H16 N4096 d128 in fp32 take 46.6 us
// (4.9 TB/s; 319 us with the rule's sum and every code decision in fp64); of B1 H32
// N16384 d128 in bf16 93.7 us (5.4 TB/s; 100.9 us with three launches, three 64-bit
// index divisions per block and two V columns per thread).  A device copy runs at
// 5.3 TB/s.
#include "gfx950.hpp"
#include "launch.hpp"

namespace fp4attn {

typedef float v2f __attribute__((ext_vector_type(2)));

// Source row of row r of the anchor-ordered matrix (Sec. "Fix 3": the anchor
// rows j * stride, j < n_anchor, first, then every other row in order);
// stride <= 1 is the identity.  Always within [0, n_anchor * stride).
template <typename I>
__device__ __forceinline__ I anchor_source_row(I r, I n_anchor, I stride) {
  if (stride <= 1) return r;
  if (r < n_anchor) return r * stride;
  const I k = r - n_anchor;
  return (k / (stride - 1)) * stride + 1 + k % (stride - 1);
}

// Source rows of consecutive anchor-ordered rows, one division for the first.
struct AnchorWalk {
  int64_t row, n_anchor, stride, src, rem;
  __device__ __forceinline__ AnchorWalk(int64_t r, int64_t n_anchor_, int64_t stride_)
      : row(r), n_anchor(n_anchor_), stride(stride_), src(r), rem(0) {
    if (stride <= 1) return;
    if (r < n_anchor) {
      src = r * stride;
    } else {
      const int64_t k = r - n_anchor, g = k / (stride - 1);
      rem = k - g * (stride - 1);
      src = g * stride + 1 + rem;
    }
  }
  __device__ __forceinline__ void next() {
    ++row;
    if (stride <= 1) {
      ++src;
    } else if (row < n_anchor) {
      src += stride;
    } else if (row == n_anchor) {  // the first row that is no anchor
      src = 1;
      rem = 0;
    } else {
      const bool skip = ++rem == stride - 1;  // over the next anchor
      src += skip ? 2 : 1;
      rem = skip ? 0 : rem;
    }
  }
};

// bf16 fast path of the same rule, exact in 32-bit arithmetic.  A bf16 value
// has at most 8 significant bits, so r = 6 v / 2^e_ceil has at most 10 and is
// exact in fp32; the hardware converter's E2M1 rounding (nearest, ties to the
// even code, saturating at 6) gives qc = E2M1(r) and qf = E2M1(2 r) exactly and
// the decode instruction returns their values, so the rule's sum is evaluated
// exactly (see below).  The codes of the chosen amplitude are the ones already
// converted (unless the E8M0 range clamps it).
//   raw[i]: elements 2i (bits 0-15) and 2i + 1 (bits 16-31).  Returns the E8M0
//   byte; codes[j] holds elements 8 j .. 8 j + 7, even element in the low nibble.
__device__ __forceinline__ unsigned mxfp4_block_bf16(const unsigned (&raw)[16], unsigned (&codes)[4]) {
  // Block maximum on the magnitude bits, two bf16 values per packed 16-bit max:
  // magnitudes order as their bit patterns, and Inf and NaN sort above every
  // finite value.
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  u16x2 mx = {0, 0};
#pragma unroll
  for (int i = 0; i < 16; ++i) mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, raw[i] & 0x7fff7fffu));
  const unsigned amax_bits = mx[0] > mx[1] ? mx[0] : mx[1];
  if (amax_bits >= 0x7f80u) {  // a NaN or an infinity in the block
#pragma unroll
    for (int j = 0; j < 4; ++j) codes[j] = 0u;
    return 255u;
  }
  // Signed values go straight into the converter: its codes carry the input's
  // sign bit (-0.0 and negative values that round to zero give 0x8).
  // encode: the codes of 6 v / 2^e, scaled in two exact steps (valid for every
  // E8M0 exponent, where the single factor 6 / 2^e may overflow).
  auto encode = [&](int e, unsigned (&w)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      unsigned acc = 0u;
      static_for<4>([&](auto P_) {
        constexpr int pb = decltype(P_)::value;
        const unsigned word = raw[4 * j + pb];
        const float v0 = __builtin_bit_cast(float, word << 16), v1 = __builtin_bit_cast(float, word & 0xffff0000u);
        acc = cvt_pk_fp4<pb>(pb == 0 ? 0u : acc, 6.0f * ldexpf(v0, -e), 6.0f * ldexpf(v1, -e), 1.0f);
      });
      w[j] = acc;
    }
  };
  if (amax_bits == 0u) {  // zero block: byte 0, every code a signed zero
    encode(0, codes);
    return 0u;
  }
  int x;
  const float m = frexpf(__builtin_bit_cast(float, amax_bits << 16), &x);  // amax = m 2^x, m in [0.5, 1)
  const int e_floor = x - 1, e_ceil = (m == 0.5f) ? x - 1 : x;
  // r = 6 v / 2^e_ceil (one exact multiply), qc = E2M1(r) and qf = E2M1(2 r)
  // (the converter divides by its scale operand and saturates at 6).  The
  // choice compares 4 sum(a r) with sum(a b), a = 2 qc - qf, b = 2 qc + qf: the
  // floor amplitude wins iff sum a (4 r - b) < 0.  Only values with |r| >= 1/8
  // have a != 0; such r are multiples of 2^-12, and |a| <= qc <= 6 because
  // qf >= qc, so both sums are exact in fp32 (multiples of 2^-13 below 2^11, and
  // of 2^-2 below 2^12).
  // The single factor 6 / 2^e_ceil is finite for e_ceil >= -125; blocks below
  // that (amax under 2^-125) take the two-step scaling of encode.
  const float sc = ldexpf(6.0f, -e_ceil);
  unsigned cc[4], cf[4];
  float s_ar = 0.0f, s_ab = 0.0f;
  auto convert = [&](auto TWO_STEP_) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      unsigned wc = 0u, wf = 0u;
      static_for<4>([&](auto P_) {
        constexpr int pb = decltype(P_)::value;
        const unsigned word = raw[4 * j + pb];
        const float v0 = __builtin_bit_cast(float, word << 16), v1 = __builtin_bit_cast(float, word & 0xffff0000u);
        float r0, r1;
        if constexpr (decltype(TWO_STEP_)::value) {
          r0 = 6.0f * ldexpf(v0, -e_ceil);
          r1 = 6.0f * ldexpf(v1, -e_ceil);
        } else {
          r0 = v0 * sc;
          r1 = v1 * sc;
        }
        wc = cvt_pk_fp4<pb>(pb == 0 ? 0u : wc, r0, r1, 1.0f);
        wf = cvt_pk_fp4<pb>(pb == 0 ? 0u : wf, r0, r1, 0.5f);
        const v2f qc = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wc, 1.0f, pb);
        const v2f qf = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wf, 1.0f, pb);
        const float a0 = fmaf(2.0f, qc[0], -qf[0]), a1 = fmaf(2.0f, qc[1], -qf[1]);
        s_ar = fmaf(a1, r1, fmaf(a0, r0, s_ar));
        s_ab = fmaf(a1, fmaf(2.0f, qc[1], qf[1]), fmaf(a0, fmaf(2.0f, qc[0], qf[0]), s_ab));
      });
      cc[j] = wc;
      cf[j] = wf;
    }
  };
  if (e_ceil >= -125) convert(std::false_type{});
  else convert(std::true_type{});
  int e = (e_floor != e_ceil && 4.0f * s_ar < s_ab) ? e_floor : e_ceil;
  e = e < -127 ? -127 : (e > 127 ? 127 : e);
  if (e == e_ceil) {
#pragma unroll
    for (int j = 0; j < 4; ++j) codes[j] = cc[j];
  } else if (e == e_floor) {
#pragma unroll
    for (int j = 0; j < 4; ++j) codes[j] = cf[j];
  } else {  // amplitude clamped to the E8M0 range
    encode(e, codes);
  }
  return (unsigned)(e + 127);
}

// MXFP8 (E4M3 payload + E8M0 per 32 values): the amplitude is the smallest
// power of two 2^e with amax / 2^e <= 448, so no payload saturates; payloads
// are v / 2^e (exact) rounded to nearest even by the hardware converter, which
// keeps E4M3 subnormals.  Zero block: u = 0; non-finite block: u = 255, codes 0.
// Codes are stored one byte per value, in the same orientation as the MXFP4
// quantizer (axis 0: transposed).
// One MXFP8 block: returns the E8M0 byte; w[i] holds the E4M3 payloads of values
// 4 i .. 4 i + 3.
__device__ __forceinline__ unsigned mxfp8_block(const float (&v)[32], unsigned (&w)[8]) {
  float amax = 0.0f;
  bool finite = true;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    finite = finite && __builtin_isfinite(v[j]);
    amax = fmaxf(amax, fabsf(v[j]));
  }
  unsigned ubyte;
  int e = 0;
  if (!finite) {
    ubyte = 255;
  } else if (amax == 0.0f) {
    ubyte = 0;
  } else {
    int x;
    frexpf(amax, &x);          // amax = m 2^x, m in [0.5, 1)
    e = x - 9;                 // amax / 2^e in [256, 512)
    if (ldexpf(amax, -e) > 448.0f) ++e;
    e = e < -127 ? -127 : (e > 127 ? 127 : e);
    ubyte = (unsigned)(e + 127);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (finite) {
      const float a0 = ldexpf(v[4 * i], -e), a1 = ldexpf(v[4 * i + 1], -e);
      const float a2 = ldexpf(v[4 * i + 2], -e), a3 = ldexpf(v[4 * i + 3], -e);
      w[i] = cvt_pk_fp8<true>(cvt_pk_fp8<false>(0u, a0, a1), a2, a3);
    } else {
      w[i] = 0u;
    }
  }
  return ubyte;
}

// The E8M0 bytes of the NB (4 or 8) blocks of group `grp` of one column (byte l of
// `run` is block NB grp + l) to `dst`: one store when every column has whole groups
// (dst is then NB-byte aligned), else one byte per block that exists.
template <int NB>
__device__ __forceinline__ void store_scale_run(uint8_t* dst, uint2 run, int64_t nblk, int64_t grp) {
  static_assert(NB == 4 || NB == 8, "one word or two");
  if (nblk % NB == 0) {
    if constexpr (NB == 8) *reinterpret_cast<uint2*>(dst) = run;
    else *reinterpret_cast<unsigned*>(dst) = run.x;
  } else {
    const uint64_t bytes = ((uint64_t)run.y << 32) | run.x;
    for (int l = 0; l < NB && grp * NB + l < nblk; ++l) dst[l] = (uint8_t)(bytes >> (8 * l));
  }
}

// fp32 form of the same rule.  r = 6 v / 2^e has up to 26 significant bits, so
// its fp32 product is rounded to odd: truncated, with the last bit set if
// anything was lost (the fma gives the product's error exactly).  Every E2M1
// boundary (of r and of 2 r) has at most three significant bits, hence an even
// last bit, so a value rounded to odd lies on the same side of each as the exact
// product and meets one only when it is exactly there: the converter's codes
// are those of the exact r.  Values under 2^-126 of the block's scale may lose
// bits in the scaling; their code is a signed zero all the same.
__device__ __forceinline__ float six_to_odd(float m) {
  const float r = 6.0f * m, err = fmaf(6.0f, m, -r);
  const unsigned lost = err != 0.0f ? 1u : 0u, over = (as_uint(err) ^ as_uint(r)) >> 31;  // |r| > |6 m|
  return as_float((as_uint(r) - (lost & over)) | lost);
}

// The rule's sum over the block in fp64, where it is exact, from the codes of
// both amplitudes.
// (The empty asm keeps the values of the common path from staying in registers
// for this rare one, and its terms in order.)
__device__ __forceinline__ bool floor_wins_f64(const float (&v)[32], int e_ceil, const unsigned (&codes_c)[4],
                                               const unsigned (&codes_f)[4]) {
  double delta = 0.0;
  unsigned cc[4], cf[4];
  static_for<16>([&](auto I_) {
    constexpr int i = decltype(I_)::value;
    if constexpr (i % 4 == 0) {
      cc[i / 4] = codes_c[i / 4];
      cf[i / 4] = codes_f[i / 4];
      asm volatile("" : "+v"(cc[i / 4]), "+v"(cf[i / 4]), "+v"(e_ceil), "+v"(delta));
    }
    const v2f qc = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(cc[i / 4], 1.0f, i % 4);
    const v2f qf = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(cf[i / 4], 1.0f, i % 4);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const double r4 = 24.0 * (double)ldexpf(v[2 * i + t], -e_ceil);
      delta += (2.0 * qc[t] - qf[t]) * (r4 - qf[t] - 2.0 * qc[t]);
    }
  });
  return delta < 0.0;
}

// One fp32 block: returns the E8M0 byte; codes as mxfp4_block_bf16.
__device__ __forceinline__ unsigned mxfp4_block_f32(const float (&v)[32], unsigned (&codes)[4]) {
  unsigned amax_bits = 0u;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    const unsigned a = as_uint(v[j]) & 0x7fffffffu;
    amax_bits = a > amax_bits ? a : amax_bits;
  }
  if (amax_bits >= 0x7f800000u) {  // a NaN or an infinity in the block
#pragma unroll
    for (int j = 0; j < 4; ++j) codes[j] = 0u;
    return 255u;
  }
  auto encode = [&](int e) {
    static_for<16>([&](auto I_) {
      constexpr int i = decltype(I_)::value;
      const float r0 = six_to_odd(ldexpf(v[2 * i], -e)), r1 = six_to_odd(ldexpf(v[2 * i + 1], -e));
      codes[i / 4] = cvt_pk_fp4<i % 4>(i % 4 == 0 ? 0u : codes[i / 4], r0, r1, 1.0f);
    });
  };
  if (amax_bits == 0u) {  // zero block: byte 0, every code a signed zero
    encode(0);
    return 0u;
  }
  int x;
  const float m = frexpf(as_float(amax_bits), &x);  // amax = m 2^x, m in [0.5, 1)
  const int e_floor = x - 1, e_ceil = (m == 0.5f) ? x - 1 : x;
  unsigned cc[4], cf[4];
  float s_ar = 0.0f, s_ab = 0.0f;
  static_for<16>([&](auto I_) {
    constexpr int i = decltype(I_)::value, w = i / 4, pb = i % 4;
    const float r0 = six_to_odd(ldexpf(v[2 * i], -e_ceil)), r1 = six_to_odd(ldexpf(v[2 * i + 1], -e_ceil));
    cc[w] = cvt_pk_fp4<pb>(pb == 0 ? 0u : cc[w], r0, r1, 1.0f);
    cf[w] = cvt_pk_fp4<pb>(pb == 0 ? 0u : cf[w], r0, r1, 0.5f);
    const v2f qc = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(cc[w], 1.0f, pb);
    const v2f qf = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(cf[w], 1.0f, pb);
    const float a0 = fmaf(2.0f, qc[0], -qf[0]), a1 = fmaf(2.0f, qc[1], -qf[1]);
    s_ar = fmaf(a1, r1, fmaf(a0, r0, s_ar));
    s_ab = fmaf(a1, fmaf(2.0f, qc[1], qf[1]), fmaf(a0, fmaf(2.0f, qc[0], qf[0]), s_ab));
    // (emits nothing: the sums are formed here and not sunk below the branch with
    // every term held in registers)
    if constexpr (pb == 3) asm volatile("" : "+v"(s_ar), "+v"(s_ab));
  });
  // s_ab is exact (see the bf16 form).  s_ar = sum a r <= 32 * 36 carries at most
  // 32 roundings of 2^-24 of it and, from each r, 2^-23: under 0.0025, so the sign
  // of 4 s_ar - s_ab stands when it is 0.0125 or more from zero.  About one block
  // in a thousand is nearer and takes the exact sum.
  bool floor_wins = false;
  if (e_floor != e_ceil) {
    const float diff = 4.0f * s_ar - s_ab;
    floor_wins = diff < 0.0f;
    if (fabsf(diff) < 0.0125f) floor_wins = floor_wins_f64(v, e_ceil, cc, cf);
  }
  int e = floor_wins ? e_floor : e_ceil;
  e = e < -127 ? -127 : (e > 127 ? 127 : e);
  if (e == e_ceil || e == e_floor) {
#pragma unroll
    for (int j = 0; j < 4; ++j) codes[j] = e == e_ceil ? cc[j] : cf[j];
  } else {  // amplitude clamped to the E8M0 range
    encode(e);
  }
  return (unsigned)(e + 127);
}

// A block of 32 values as the block functions take it: bf16 pairs in 16 words,
// fp32 values as they are.
template <typename T>
struct Block;
template <>
struct Block<uint16_t> {
  unsigned raw[16];
  __device__ __forceinline__ unsigned mxfp4(unsigned (&w)[4]) const { return mxfp4_block_bf16(raw, w); }
  __device__ __forceinline__ unsigned mxfp8(unsigned (&w)[8]) const {
    float v[32];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      v[2 * i] = as_float(raw[i] << 16);
      v[2 * i + 1] = as_float(raw[i] & 0xffff0000u);
    }
    return mxfp8_block(v, w);
  }
  // element j from a value in memory (j in order, even first)
  __device__ __forceinline__ void set(int j, uint16_t x) {
    if (j % 2 == 0) raw[j / 2] = x;
    else raw[j / 2] |= (unsigned)x << 16;
  }
};
template <>
struct Block<float> {
  float v[32];
  __device__ __forceinline__ unsigned mxfp4(unsigned (&w)[4]) const { return mxfp4_block_f32(v, w); }
  __device__ __forceinline__ unsigned mxfp8(unsigned (&w)[8]) const { return mxfp8_block(v, w); }
  __device__ __forceinline__ void set(int j, float x) { v[j] = x; }
};

// 32 contiguous values (16-byte aligned).
template <typename T>
__device__ __forceinline__ void load_row_block(const T* p, Block<T>& b) {
  constexpr int kLoads = 32 * sizeof(T) / 16;
  uint4 q[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; ++i) q[i] = reinterpret_cast<const uint4*>(p)[i];
  static_assert(sizeof(b) == sizeof(q), "a block is its values' bytes");
  __builtin_memcpy(&b, q, sizeof(q));
}

// Blocks along the contiguous axis (Q, K): `total` blocks of `nblk` per row.
struct RowsJob {
  const void* src;
  uint8_t* codes;
  uint8_t* scales;
  int64_t total, rows, nblk, n_anchor, stride;  // stride > 1: rows in anchor order
};
// Blocks along rows, output transposed (V): `batch` matrices of rows x cols.
struct ColsJob {
  const void* src;
  uint8_t* codes;
  uint8_t* scales;
  int64_t rows, cols, n_anchor, stride;
};

constexpr int kThreads = 512;     // one block of 32 values per thread (the joint launch)
constexpr int kColsPerWg = 64;    // V: 64 columns x one block of 32 rows per wave

// Without the anchor order block t is at value 32 t: no division.
template <typename T, int NT>
__device__ __forceinline__ void quantize_rows(const RowsJob& j, unsigned wg) {
  const int64_t t = (int64_t)wg * NT + threadIdx.x;
  if (t >= j.total) return;
  const T* src = static_cast<const T*>(j.src);
  int64_t at = t;
  if (j.stride > 1) {
    if (j.total <= 0x7fffffff) {
      const unsigned row = (unsigned)t / (unsigned)j.nblk, b = row / (unsigned)j.rows;
      const unsigned o = row - b * (unsigned)j.rows;
      at = (int64_t)(b * (unsigned)j.rows + anchor_source_row<unsigned>(o, j.n_anchor, j.stride)) * j.nblk +
           ((unsigned)t - row * (unsigned)j.nblk);
    } else {
      const int64_t row = t / j.nblk, b = row / j.rows;
      at = (b * j.rows + anchor_source_row<int64_t>(row - b * j.rows, j.n_anchor, j.stride)) * j.nblk + (t - row * j.nblk);
    }
  }
  Block<T> blk;
  load_row_block(src + at * 32, blk);
  unsigned w[4];
  const unsigned u = blk.mxfp4(w);
  *reinterpret_cast<v4i*>(j.codes + t * 16) = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
  j.scales[t] = (uint8_t)u;
}

// Staged V^T: a workgroup of NT threads takes 64 columns x NT / 2 rows, wave w block w
// of their 32-row blocks.  fp32: lane = column, 256-byte row segments.  bf16: lane l < 32 reads
// rows 0-15 of the block at columns 2 l and 2 l + 1, lane l + 32 rows 16-31, and
// one exchange of the wave's halves leaves column 2 l in lane l and column
// 2 l + 1 in lane l + 32.  Codes and scale bytes are parked in LDS (chunks XOR'd
// with the column, so that neither side meets bank conflicts) and leave as one
// contiguous run per column (128 bytes for 512 threads, MXFP8 256) and one scale store.  The
// workgroups of the column groups of the same rows are launched next to each
// other, so wider rows are read whole at about the same time.  cols % 64 == 0;
// blocks past the last are skipped (their waves still meet the barrier).
template <typename T, bool FP8, int NT>
__device__ __forceinline__ void quantize_cols(const ColsJob& j, unsigned wg) {
  constexpr int kBlksPerWg = NT / kColsPerWg;                 // blocks of 32 rows, one per wave
  constexpr int kChunks = FP8 ? 2 * kBlksPerWg : kBlksPerWg;  // 16-byte chunks of a column's run
  __shared__ uint4 code_lds[kColsPerWg][kChunks];
  __shared__ uint2 scale_lds[kColsPerWg];  // 8 bytes a column, the first kBlksPerWg used
  const unsigned nblk = (unsigned)(j.rows / 32), ngrp = (nblk + kBlksPerWg - 1) / kBlksPerWg;
  const unsigned ncg = (unsigned)(j.cols / kColsPerWg);
  const unsigned rest = wg / ncg, cg = wg - rest * ncg, b = rest / ngrp, grp = rest - b * ngrp;
  const int tid = threadIdx.x, lane = tid & 63, lb = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t blk = (int64_t)grp * kBlksPerWg + lb;
  if (blk < nblk) {
    const T* base = static_cast<const T*>(j.src) + (int64_t)b * j.rows * j.cols + cg * kColsPerWg;
    Block<T> bl;
    int c;  // this lane's column of the 64
    if constexpr (sizeof(T) == 2) {
      const int cp = lane & 31, half = lane >> 5;
      c = 2 * cp + half;
      unsigned pair[16];
      const T* p = base + 2 * cp;
      if (j.stride > 1) {
        AnchorWalk r(blk * 32 + 16 * half, j.n_anchor, j.stride);
#pragma unroll
        for (int i = 0; i < 16; ++i, r.next()) pair[i] = *reinterpret_cast<const unsigned*>(p + r.src * j.cols);
      } else {
        p += (blk * 32 + 16 * half) * j.cols;
#pragma unroll
        for (int i = 0; i < 16; ++i) pair[i] = *reinterpret_cast<const unsigned*>(p + i * j.cols);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        unsigned even = (pair[2 * i] & 0xffffu) | (pair[2 * i + 1] << 16);         // column 2 cp, two rows
        unsigned odd = (pair[2 * i] >> 16) | (pair[2 * i + 1] & 0xffff0000u);      // column 2 cp + 1
        swap_halves(even, odd);
        bl.raw[i] = even;
        bl.raw[8 + i] = odd;
      }
    } else {
      c = lane;
      const T* p = base + lane;
      if (j.stride > 1) {
        AnchorWalk r(blk * 32, j.n_anchor, j.stride);  // wave-uniform
#pragma unroll
        for (int i = 0; i < 32; ++i, r.next()) bl.set(i, p[r.src * j.cols]);
      } else {
        p += blk * 32 * j.cols;
#pragma unroll
        for (int i = 0; i < 32; ++i) bl.set(i, p[i * j.cols]);
      }
    }
    uint8_t* sb = reinterpret_cast<uint8_t*>(scale_lds);
    if constexpr (FP8) {
      unsigned w[8];
      sb[8 * c + lb] = (uint8_t)bl.mxfp8(w);
      code_lds[c][(2 * lb) ^ (c & (kChunks - 1))] = uint4{w[0], w[1], w[2], w[3]};
      code_lds[c][(2 * lb + 1) ^ (c & (kChunks - 1))] = uint4{w[4], w[5], w[6], w[7]};
    } else {
      unsigned w[4];
      sb[8 * c + lb] = (uint8_t)bl.mxfp4(w);
      code_lds[c][lb ^ (c & (kChunks - 1))] = uint4{w[0], w[1], w[2], w[3]};
    }
  }
  __syncthreads();
  // kBlksPerWg lanes write a column's run, 16 bytes each at a time
  const int c = tid / kBlksPerWg;
  const int64_t col = (int64_t)b * j.cols + cg * kColsPerWg + c;
  constexpr int kBlkChunks = FP8 ? 2 : 1;
  uint8_t* cdst = j.codes + (col * nblk + (int64_t)grp * kBlksPerWg) * (16 * kBlkChunks);
#pragma unroll
  for (int k = 0; k < kBlkChunks; ++k) {
    const int ch = tid % kBlksPerWg + kBlksPerWg * k;
    if (grp * kBlksPerWg + ch / kBlkChunks < nblk)
      *reinterpret_cast<uint4*>(cdst + ch * 16) = code_lds[c][ch ^ (c & (kChunks - 1))];
  }
  if (tid < kColsPerWg)
    store_scale_run<kBlksPerWg>(j.scales + ((int64_t)b * j.cols + cg * kColsPerWg + tid) * nblk + grp * kBlksPerWg, scale_lds[tid],
                    nblk, grp);
}

template <typename T, int NT>
__global__ __launch_bounds__(NT) void quantize_mxfp4_rows_kernel(const RowsJob j) {
  quantize_rows<T, NT>(j, blockIdx.x);
}
template <typename T, bool FP8, int NT>
__global__ __launch_bounds__(NT) void quantize_cols_kernel(const ColsJob j) {
  quantize_cols<T, FP8, NT>(j, blockIdx.x);
}

// Q, K and V in one launch: workgroups [0, n_v) take V (the longest of the three
// for a small call), the next n_q Q, the rest K.  One launch instead of three, and
// the three fill the chip together: bf16 B3 H10 N1920 d64 21.7 us in three kernels,
// 10.0 us in one; B1 H32 N16384 d128 99.2 -> 93.7 us; fp32 B2 H16 N4096 d128
// 54.7 -> 46.6 us.
template <typename T, bool FP8>
__global__ __launch_bounds__(kThreads) void quantize_qkv_kernel(const RowsJob q, const RowsJob k, const ColsJob v,
                                                                unsigned n_v, unsigned n_q) {
  const unsigned wg = blockIdx.x;
  if (wg < n_v) quantize_cols<T, FP8, kThreads>(v, wg);
  else if (wg < n_v + n_q) quantize_rows<T, kThreads>(q, wg - n_v);
  else quantize_rows<T, kThreads>(k, wg - n_v - n_q);
}

// MXFP4, blocks along rows with transposed output, any number of columns: a
// thread takes one block, consecutive threads consecutive columns.
template <typename T>
__global__ __launch_bounds__(256) void quantize_mxfp4_cols_any_kernel(const T* __restrict__ src, int64_t batch,
                                                                      int64_t rows, int64_t cols,
                                                                      uint8_t* __restrict__ codes,
                                                                      uint8_t* __restrict__ scales, int64_t n_anchor,
                                                                      int64_t anchor_stride) {
  const int64_t nblk = rows / 32;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= batch * cols * nblk) return;
  const int64_t c = t % cols, blk = (t / cols) % nblk, b = t / (cols * nblk);
  const T* p = src + b * rows * cols + c;
  Block<T> bl;
  AnchorWalk r(blk * 32, n_anchor, anchor_stride);
#pragma unroll
  for (int i = 0; i < 32; ++i, r.next()) bl.set(i, p[r.src * cols]);
  unsigned w[4];
  scales[(b * cols + c) * nblk + blk] = (uint8_t)bl.mxfp4(w);
  *reinterpret_cast<v4i*>(codes + ((b * cols + c) * nblk + blk) * 16) = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
}

// bf16, blocks along rows with transposed output (V): a thread takes one block
// of two adjacent columns (one 4-byte load per row; a wave reads 256-byte row
// segments).  cols % 2 == 0.  (Several blocks per thread, for longer runs of
// contiguous code bytes, measured slower: fewer waves in flight.)
__global__ __launch_bounds__(256) void quantize_mxfp4_bf16_cols_kernel(const uint16_t* __restrict__ src, int64_t batch,
                                                                       int64_t rows, int64_t cols,
                                                                       uint8_t* __restrict__ codes,
                                                                       uint8_t* __restrict__ scales, int64_t n_anchor,
                                                                       int64_t anchor_stride) {
  const int64_t nblk = rows / 32, npair = cols / 2;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= batch * nblk * npair) return;
  const int64_t cp = t % npair, blk = (t / npair) % nblk, b = t / (npair * nblk);
  const uint16_t* base = src + b * rows * cols + 2 * cp;
  unsigned pair[32];
  AnchorWalk r(blk * 32, n_anchor, anchor_stride);
#pragma unroll
  for (int j = 0; j < 32; ++j, r.next()) pair[j] = *reinterpret_cast<const unsigned*>(base + r.src * cols);
  unsigned raw0[16], raw1[16];  // column 2 cp and 2 cp + 1, rows in order
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    raw0[i] = (pair[2 * i] & 0xffffu) | (pair[2 * i + 1] << 16);
    raw1[i] = (pair[2 * i] >> 16) | (pair[2 * i + 1] & 0xffff0000u);
  }
  const int64_t col0 = b * cols + 2 * cp;
  unsigned w[4];
  scales[col0 * nblk + blk] = (uint8_t)mxfp4_block_bf16(raw0, w);
  *reinterpret_cast<v4i*>(codes + (col0 * nblk + blk) * 16) = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
  scales[(col0 + 1) * nblk + blk] = (uint8_t)mxfp4_block_bf16(raw1, w);
  *reinterpret_cast<v4i*>(codes + ((col0 + 1) * nblk + blk) * 16) = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
}

template <typename T>
__device__ __forceinline__ float load_as_float(const T* p);
template <>
__device__ __forceinline__ float load_as_float<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float load_as_float<uint16_t>(const uint16_t* p) {
  return __builtin_bit_cast(float, (unsigned)(*p) << 16);
}

template <typename T, int AXIS>
__global__ __launch_bounds__(256) void quantize_mxfp8_kernel(const T* __restrict__ src, int64_t batch, int64_t rows,
                                                             int64_t cols, uint8_t* __restrict__ codes,
                                                             uint8_t* __restrict__ scales) {
  const int64_t nblk = AXIS == 1 ? cols / 32 : rows / 32;
  const int64_t outer = AXIS == 1 ? rows : cols;
  const int64_t total = batch * outer * nblk;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  int64_t b, o, blk;
  if (AXIS == 1) {
    blk = t % nblk;
    o = (t / nblk) % outer;
    b = t / (nblk * outer);
  } else {
    o = t % outer;
    blk = (t / outer) % nblk;
    b = t / (outer * nblk);
  }
  float v[32];
  if (AXIS == 1) {
    const T* p = src + (b * rows + o) * cols + blk * 32;
#pragma unroll
    for (int j = 0; j < 32; ++j) v[j] = load_as_float<T>(p + j);
  } else {
    const T* p = src + (b * rows + blk * 32) * cols + o;
#pragma unroll
    for (int j = 0; j < 32; ++j) v[j] = load_as_float<T>(p + (int64_t)j * cols);
  }
  unsigned w[8];
  const unsigned ubyte = mxfp8_block(v, w);
  uint8_t* cdst = codes + (b * outer + o) * (nblk * 32) + blk * 32;
  *reinterpret_cast<v4i*>(cdst) = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
  *reinterpret_cast<v4i*>(cdst + 16) = v4i{(int)w[4], (int)w[5], (int)w[6], (int)w[7]};
  scales[(b * outer + o) * nblk + blk] = (uint8_t)ubyte;
}

namespace {

template <int NT>
int64_t workgroups(const RowsJob& j) { return (j.total + NT - 1) / NT; }
template <int NT>
int64_t workgroups(const ColsJob& j, int64_t batch) {
  constexpr int kBlks = NT / kColsPerWg;
  return batch * (j.cols / kColsPerWg) * ((j.rows / 32 + kBlks - 1) / kBlks);
}

template <typename T, int NT>
hipError_t launch_rows_nt(const RowsJob& j, hipStream_t stream) {
  hipLaunchKernelGGL((quantize_mxfp4_rows_kernel<T, NT>), dim3((unsigned)workgroups<NT>(j)), dim3(NT), 0, stream, j);
  return hipGetLastError();
}

// Rows in a launch of their own: 256 threads up to 327680 blocks, where workgroups of 512
// leave the chip half filled or a round half empty (us, 256 / 512: bf16 1024 rows of 64
// 2.94 / 3.46, 11 x 3968 rows of 128 4.41 / 5.00, 256 x 384 of 96 5.79 / 6.36; fp32 4.31 /
// 5.02, 7.25 / 8.43); above, 512 is even (bf16 22 x 3968 of 128 6.51 / 6.57) or ahead (fp32
// 11.7 / 11.1).
template <typename T>
hipError_t launch_rows(const RowsJob& j, hipStream_t stream) {
  return j.total <= 5 << 16 ? launch_rows_nt<T, 256>(j, stream) : launch_rows_nt<T, kThreads>(j, stream);
}

// A launch holds fewer than 2^32 threads; more matrices than that take several.
template <int NT>
constexpr int64_t kMaxWorkgroups = (int64_t(1) << 32) / NT - 1;

template <typename T, bool FP8, int NT>
hipError_t launch_cols_nt(ColsJob j, int64_t batch, hipStream_t stream) {
  const int64_t per = workgroups<NT>(j, 1), fit = kMaxWorkgroups<NT> / per, chunk = fit > 1 ? fit : 1;
  const int64_t values = j.rows * j.cols;
  for (int64_t b = 0; b < batch; b += chunk) {
    const int64_t n = batch - b < chunk ? batch - b : chunk;
    hipLaunchKernelGGL((quantize_cols_kernel<T, FP8, NT>), dim3((unsigned)(n * per)), dim3(NT), 0, stream, j);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    j.src = static_cast<const T*>(j.src) + n * values;
    j.codes += n * (FP8 ? values : values / 2);
    j.scales += n * (values / 32);
  }
  return hipSuccess;
}

// V^T in a launch of its own: 256 threads up to 196608 blocks, where a grid of 512 leaves
// the chip half filled or starts a round it does not fill (us, 256 / 512: 2 x 1024 rows of
// 64, bf16 MXFP4 3.60 / 4.08, fp32 MXFP8 3.55 / 3.72; 11 x 3968 rows of 128 5.16 / 6.09,
// 4.99 / 5.65), and for bf16 MXFP4 on every size (48 x 4096 rows of 128 14.5 / 16.1, 32 x
// 16384 32.9 / 33.5).  The other types gain from the longer runs of 512 (24 x 4096 rows of
// 128: fp32 MXFP4 13.7 / 12.35, MXFP8 11.25 / 10.6; 48 x 4096: bf16 MXFP8 14.6 / 13.9).
template <typename T, bool FP8>
hipError_t launch_cols(const ColsJob& j, int64_t batch, hipStream_t stream) {
  const bool small = (sizeof(T) == 2 && !FP8) || batch * j.cols * (j.rows / 32) <= 3 << 16;
  return small ? launch_cols_nt<T, FP8, 256>(j, batch, stream) : launch_cols_nt<T, FP8, kThreads>(j, batch, stream);
}

template <typename T, bool FP8>
hipError_t launch_qkv(const RowsJob& q, const RowsJob& k, const ColsJob& v, int64_t batch, hipStream_t stream) {
  const unsigned n_v = (unsigned)workgroups<kThreads>(v, batch), n_q = (unsigned)workgroups<kThreads>(q);
  hipLaunchKernelGGL((quantize_qkv_kernel<T, FP8>), dim3(n_v + 2 * n_q), dim3(kThreads), 0, stream, q, k, v, n_v, n_q);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_quantize_mxfp4(const void* src, int src_dtype, int64_t batch, int64_t rows, int64_t cols, int axis,
                                 int64_t n_anchor, uint8_t* codes, uint8_t* scales, hipStream_t stream) {
  const int64_t stride = n_anchor > 0 ? rows / n_anchor : 0;
  const bool bf16 = src_dtype == 1;
  if (axis == 1) {
    const RowsJob j{src, codes, scales, batch * rows * (cols / 32), rows, cols / 32, n_anchor, stride};
    return bf16 ? launch_rows<uint16_t>(j, stream) : launch_rows<float>(j, stream);
  }
  if (cols % kColsPerWg == 0) {  // whole column groups; otherwise lanes of the staged kernel would idle
    const ColsJob j{src, codes, scales, rows, cols, n_anchor, stride};
    return bf16 ? launch_cols<uint16_t, false>(j, batch, stream) : launch_cols<float, false>(j, batch, stream);
  }
  const int64_t nblk = rows / 32;
  const bool pairs = bf16 && cols % 2 == 0;  // two columns per thread, 4-byte loads
  const int64_t threads = batch * nblk * (pairs ? cols / 2 : cols);
  const dim3 grid((unsigned)((threads + 255) / 256)), block(256);
  if (pairs)
    hipLaunchKernelGGL(quantize_mxfp4_bf16_cols_kernel, grid, block, 0, stream, (const uint16_t*)src, batch, rows, cols,
                       codes, scales, n_anchor, stride);
  else if (bf16)
    hipLaunchKernelGGL((quantize_mxfp4_cols_any_kernel<uint16_t>), grid, block, 0, stream, (const uint16_t*)src, batch,
                       rows, cols, codes, scales, n_anchor, stride);
  else
    hipLaunchKernelGGL((quantize_mxfp4_cols_any_kernel<float>), grid, block, 0, stream, (const float*)src, batch, rows,
                       cols, codes, scales, n_anchor, stride);
  return hipGetLastError();
}

hipError_t launch_quantize_mxfp8(const void* src, int src_dtype, int64_t batch, int64_t rows, int64_t cols, int axis,
                                 uint8_t* codes, uint8_t* scales, hipStream_t stream) {
  const bool bf16 = src_dtype == 1;
  if (axis == 0 && cols % kColsPerWg == 0) {
    const ColsJob j{src, codes, scales, rows, cols, 0, 0};
    return bf16 ? launch_cols<uint16_t, true>(j, batch, stream) : launch_cols<float, true>(j, batch, stream);
  }
  const int64_t nblk = axis == 1 ? cols / 32 : rows / 32;
  const int64_t outer = axis == 1 ? rows : cols;
  const int64_t total = batch * outer * nblk;
  const dim3 grid((unsigned)((total + 255) / 256)), block(256);
  if (!bf16) {
    if (axis == 1)
      hipLaunchKernelGGL((quantize_mxfp8_kernel<float, 1>), grid, block, 0, stream, (const float*)src, batch, rows,
                         cols, codes, scales);
    else
      hipLaunchKernelGGL((quantize_mxfp8_kernel<float, 0>), grid, block, 0, stream, (const float*)src, batch, rows,
                         cols, codes, scales);
  } else {
    if (axis == 1)
      hipLaunchKernelGGL((quantize_mxfp8_kernel<uint16_t, 1>), grid, block, 0, stream, (const uint16_t*)src, batch,
                         rows, cols, codes, scales);
    else
      hipLaunchKernelGGL((quantize_mxfp8_kernel<uint16_t, 0>), grid, block, 0, stream, (const uint16_t*)src, batch,
                         rows, cols, codes, scales);
  }
  return hipGetLastError();
}

hipError_t launch_quantize_qkv(const QkvArgs& a, hipStream_t stream) {
  // one launch where V takes the staged kernel and the three fit one; otherwise one
  // launch each
  const int64_t total = a.batch * a.rows * (a.cols / 32), stride = a.n_anchor > 0 ? a.rows / a.n_anchor : 0;
  const RowsJob q{a.q, a.q_codes, a.q_scales, total, a.rows, a.cols / 32, 0, 0};
  const RowsJob k{a.k, a.k_codes, a.k_scales, total, a.rows, a.cols / 32, a.n_anchor, stride};
  const ColsJob v{a.v, a.vt_codes, a.vt_scales, a.rows, a.cols, a.n_anchor, stride};
  if (a.cols % kColsPerWg != 0 || workgroups<kThreads>(v, a.batch) + 2 * workgroups<kThreads>(q) > kMaxWorkgroups<kThreads>) {
    hipError_t e = launch_quantize_mxfp4(a.q, a.src_dtype, a.batch, a.rows, a.cols, 1, 0, a.q_codes, a.q_scales, stream);
    if (e != hipSuccess) return e;
    e = launch_quantize_mxfp4(a.k, a.src_dtype, a.batch, a.rows, a.cols, 1, a.n_anchor, a.k_codes, a.k_scales, stream);
    if (e != hipSuccess) return e;
    return a.v_fp8 ? launch_quantize_mxfp8(a.v, a.src_dtype, a.batch, a.rows, a.cols, 0, a.vt_codes, a.vt_scales, stream)
                   : launch_quantize_mxfp4(a.v, a.src_dtype, a.batch, a.rows, a.cols, 0, a.n_anchor, a.vt_codes,
                                           a.vt_scales, stream);
  }
  if (a.src_dtype == 1)
    return a.v_fp8 ? launch_qkv<uint16_t, true>(q, k, v, a.batch, stream) : launch_qkv<uint16_t, false>(q, k, v, a.batch, stream);
  return a.v_fp8 ? launch_qkv<float, true>(q, k, v, a.batch, stream) : launch_qkv<float, false>(q, k, v, a.batch, stream);
}

}  // namespace fp4attn
