// Which workgroup shape a forward launches.  Plain C++, so that a host program can ask
// the rules what a launch takes.
#pragma once
#include <cstdint>

namespace fp4attn {

// A workgroup's shape: qg query tiles of 32, ks key groups (ks = 1: every wave
// walks all keys).
struct Shape {
  int qg, ks;
};

// The shape of a launch, from U = workgroups of 128 queries and W = workgroups of
// 256 (0 where N is no multiple of 256), against 256 CUs.
//
// A key split multiplies the workgroups (half: eight waves per 128 queries,
// quarter: per 64, eighth: per 32) and divides the serial steps of a wave; it copies
// K and V 2, 4 or 8 times as often per query as a wide workgroup.  It pays while its
// workgroups do not exceed the CUs and the loop is longer than the merge.  Measured
// per launch (graph replays, us; narrow / wide / half / quarter / eighth):
//   d 128  U 32 N 4096   29.7 / 40.2 / 26.0 / 18.9 / 15.7    U 64 N 512   8.8 / 11.4 / 9.3 / 8.2 / 7.6
//          U 128 N 4096  31.0 / 41.3 / 27.1 / 21.3 / 31.6    U 128 N 512  9.4 / 12.0 / 9.9 / 9.0 / 13.5
//          U 192 N 2048  19.5 / 25.1 / 18.4 / 25.6 / 30.5    U 192 N 1024 13.2 / 16.9 / 13.2 / 19.1 / 23.5
//   d 64   U 64 N 2048   15.4 / 19.5 / 13.1 / 9.8 / 9.3      U 64 N 512   6.7 / 8.3 / 7.1 / 6.1 / 6.5
//          U 256 N 1024  10.6 / 12.9 / 10.3 / 14.0 / 24.9    U 512 N 4096 37.7 / 36.5 / 34.9 / 53.0 / 90.2
// The causal forward's workgroups are half as long on average and unequal, so its
// splits pay further: d 128 N 4096 U 192 31.8 / 42.9 / 27.8 / 24.1 / 34.4, U 512 38.2 / 44.8
// / 36.6 / 52.2; d 64 N 2048 U 448 17.9 / 22.3 / 17.0 / 26.8; but N 1024 U 384 d 128 16.0 / 19.7
// / 19.3, and below N 512 half never gains on narrow (narrow / half: d 128 N 128 U 8 6.5 / 7.1,
// N 256 U 32 7.5 / 8.0; d 64 N 128 U 32 5.3 / 5.6, N 256 U 64 6.1 / 6.3).
// FP8 P/V with d = 128 leaves one wave per SIMD to four-wave workgroups (LDS):
// N 4096 U 128 52.6 / 65.9 / 38.8 / 26.3, U 256 54.5 / 67.0 / 42.8 / 48.0.
// The guarded and exponential routes share the plain lines: (110, 16) and 16 of 16 pairs,
// d 128 N 4096 U 32 31.0 / 41.6 / 25.6 / 17.9 / 15.5 and 37.2 / 56.4 / 32.7 / 21.7 / 16.8, U 128
// 32.2 / 42.7 / 27.7 / 21.5 / 32.6 and 38.9 / 57.9 / 35.3 / 25.6 / 35.5, U 256 34.8 / 44.0 / 30.9 /
// 39.0 / 60.0 and 41.0 / 58.8 / 37.5 / 45.9 / 64.7, U 384 48.9 / 44.7 / 54.8 and 61.9 / 59.6 / 68.4, U 768
// 79.2 / 89.3 / 83.7 and 93.1 / 114.8 / 102.4; d 64 N 4096 U 512 38.8 / 38.4 / 36.1 and 52.9 / 52.3 /
// 49.0.  Over 183 grids of N 512 to 8192 the rule's shape takes 0.2 % (guard), 0.4 % (4 pairs) and
// 0.6 % (16) longer than the fastest on geometric mean; the most, 8 to 11 %, at N 512 and
// U 1024 to 3072, where narrow is ahead of wide on the plain route too.
inline Shape directp_shape(int d, int N, int bh, bool causal, bool fp8) {
  const int64_t U = (int64_t)bh * (N / 128), W = N % 256 == 0 ? U / 2 : 0;
  const Shape narrow{4, 1}, wide{8, 1}, half{4, 2}, quarter{2, 4}, eighth{1, 8};
  const bool fp8_128 = fp8 && d == 128;  // (its eighth does not fit the LDS)
  if (U <= 64 && N >= (d == 64 ? 1024 : 512) && !fp8_128) return eighth;
  if (U <= 128 && N >= 512) return quarter;
  if (causal && N >= 4096 && U <= (d == 64 || fp8 ? 256 : 192)) return quarter;
  if (U <= 256 && N >= (d == 64 || causal || fp8 ? 1024 : 2048)) return half;
  if (fp8_128) {
    // Whole rounds favour wide workgroups (N 4096 U 512 70.7 against 80.8 us); half takes
    // a second round that wide would leave half empty (U 640 114.8 / 132.5, U 768 120.3 /
    // 132.9), unequal workgroups (causal U 320 40.1 / 66.3, U 512 48.8 / 67.4), and every
    // N that 256 does not divide (N 3968 U 744 110.9 against narrow's 148.0).  Not below
    // N 1024 (half / wide: 44.8 / 46.1 there for U 544, but N 768 U 702 46.9 / 40.4, N 512
    // U 768 35.8 / 32.1, N 256 U 768 29.5 / 25.6; causal N 256 U 512 19.4 / 16.5, N 512 U 512
    // 21.9 / 19.4, U 384 18.6 / 18.6, U 288 15.8 / 17.6).
    const bool split = causal ? U <= (N >= 1024 ? 512 : 384) : W > 256 && W <= 384 && N >= 1024;
    if (W == 0 || split) return half;
    return W > 128 ? wide : narrow;
  }
  if (fp8) {
    // d = 64: narrow workgroups, two per CU, throughout (N 4096 U 768 81.1 against wide's
    // 106.6, U 4096 376 / 418).
    return causal && N >= 512 && U <= 512 && U <= N / 8 ? half : narrow;
  }
  if (d == 64) {
    // Four waves per SIMD (one-step pipeline).  Wide workgroups, two per CU, for whole
    // half rounds (+4-8 % on large shapes; -6 to -15 % where the last is partly
    // filled) and, causal, from 3072 of them (+2.5-5.7 %; -1 to -2 % at 1024-2048).
    if (causal ? N >= 512 && U <= 640 && U <= N / 4 : U <= 512 && N >= 2048) return half;
    return W >= (causal ? 3072 : 256) && W % 256 == 0 ? wide : narrow;
  }
  if (causal) {
    // Wide from a round and a half on for long rows (N 4096 U 768 47.8 against 49.6, U 896
    // 55.0 / 56.3, U 1024 57.0 / 58.9, U 4096 238 / 247; N 8192 U 768 82.5 / 82.9, U 896 89.4 / 98.0,
    // U 1024 95.2 / 103.4), but not below (N 4096 U 640 45.9 / 41.1), nor between two rounds
    // and four (N 4096 U 1280 78.4 / 71.9, U 1536 90.0 / 84.9; N 8192 U 1280 132.1 / 127.7), and never for short rows (N 2048 U 512 28.4 / 23.4, U 4096
    // 175 / 172; N 1024 U 1024 33.3 / 30.7).
    if (N >= 512 && U <= 512 && U <= N / 8) return half;
    return N >= 4096 && ((W >= 384 && W <= 512) || W >= 1024) ? wide : narrow;
  }
  // Wide when more than half the CUs get one (N 4096 U 384 43.1 against 46.4, U 448 44.7 /
  // 48.5; N 512 even), except where the grid takes two to five rounds and the last is
  // at most half full: narrow workgroups, two per CU, finish that tail sooner (N 4096
  // U 768 78.3 / 85.4; at ten rounds 2 % slower).
  const bool tail = W > 256 && W <= 5 * 256 && W % 256 != 0 && W % 256 <= 128;
  return W > (N >= 1024 ? 128 : 255) && !tail ? wide : narrow;
}

// Whether directp_shape ever returns `s`: a kernel is built for these only.  FP8 P/V with
// d = 64 takes no wide workgroups; with d = 128 its eighth does not fit the LDS, and its
// causal form splits every grid that wide workgroups do not fill.
constexpr bool directp_launches(int d, bool causal, bool fp8, Shape s) {
  const bool wide = s.qg == 8, narrow = s.qg == 4 && s.ks == 1;
  return !fp8 || (d == 64 ? !wide : s.ks != 8 && !(causal && narrow));
}

// The same for the BF16 forward (U and W as above).  Wide: 256
// queries, eight waves; half: 128 queries, eight waves, the keys split in two;
// narrow: 128 queries, four waves (with d = 128 one wave per SIMD, since its ring
// fills the LDS).  Measured per launch (us, narrow / wide / half):
//   d 128 N 4096  U 128 81.0 / 102.4 / 60.7   U 384 161.6 / 110.8 / 128.6   U 640 242.3 / 228.0 / 199.3
//                 U 768 234.0 / 218.6 / 201.1   U 896 307.3 / 225.6 / 252.8   U 1024 333.2 / 260.1 / 282.2;  N 1024 U 768 79.6 / 70.9 / 72.2;  N 3968 U 744 239.6 / - / 202.7
//   d 64  N 4096  U 128 46.3 / 65.1 / 39.8    U 384 72.3 / 67.6 / 69.2      U 640 116.0 / 121.8 / 108.7
//                 U 896 149.3 / 134.0 / 144.2;  N 512 U 256 10.7 / 13.8 / 11.0, U 640 23.0 / 24.5 / 23.6
inline Shape bf16_shape(int d, int N, int bh) {
  const int64_t U = (int64_t)bh * (N / 128), W = N % 256 == 0 ? U / 2 : 0;
  bool wide, half;
  if (d == 128) {
    // half where its workgroups fit the CUs, where wide ones would leave a second
    // round half empty, and wherever wide ones do not exist
    half = N >= 512 && (U <= 256 || W == 0 || (W > 256 && W <= 384 && N >= 2048));
    wide = !half && W > 128;
  } else {
    // likewise, two workgroups per CU
    const bool second = U > 512 && U <= 768;
    half = N >= 1024 && (U <= 256 || second || (W == 0 && U <= 768));
    wide = !half && W > 128 && !second;
  }
  return half ? Shape{4, 2} : Shape{wide ? 8 : 4, 1};
}

}  // namespace fp4attn
