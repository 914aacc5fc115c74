// Direct-P full-MXFP4 attention forward: host dispatch (the kernel and its
// design are in fwd_mxfp4.hpp).  The EX2 = 0 variants are compiled here; the
// native-exponential densities come from fwd_mxfp4_ex2*.hip, the guarded
// variants from fwd_mxfp4_guard.hip and the causal ones from
// fwd_mxfp4_causal.hip, the FP8 P/V route from fwd_mxfp4_fp8pv.hip, all
// compiled in parallel with this file.
#include "fwd_mxfp4.hpp"

namespace fp4attn {
namespace directp_detail {

FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DEFINE, 0, kVarOnline)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 1, kVarOnline)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 2, kVarOnline)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 4, kVarOnline)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 8, kVarOnline)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 16, kVarOnline)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 0, kVarGuard)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 4, kVarGuard)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 16, kVarGuard)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 0, kVarCausal)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 4, kVarCausal)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 16, kVarCausal)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 0, kVarOnline | kPV8)
FP4ATTN_DIRECTP_VARIANTS(FP4ATTN_DIRECTP_DECLARE, 0, kVarCausal | kPV8)

namespace {

// The guarded and causal variants exist for the densities 0, 4 and 16.
template <int D, int QG, int KS, bool DUMP, int VAR>
hipError_t dispatch_ex2_subset(const KParams& kp, int ex2, hipStream_t stream) {
  switch (ex2) {
    case 0: return launch_directp<D, QG, KS, DUMP, 0, VAR>(kp, stream);
    case 4: return launch_directp<D, QG, KS, DUMP, 4, VAR>(kp, stream);
    case 16: return launch_directp<D, QG, KS, DUMP, 16, VAR>(kp, stream);
    default: return hipErrorInvalidValue;
  }
}

template <int D, int QG, int KS, bool DUMP>
hipError_t dispatch_ex2(const KParams& kp, int ex2, int var, hipStream_t stream) {
  if (var == (kVarOnline | kPV8)) return launch_directp<D, QG, KS, DUMP, 0, kVarOnline | kPV8>(kp, stream);
  if (var == (kVarCausal | kPV8)) return launch_directp<D, QG, KS, DUMP, 0, kVarCausal | kPV8>(kp, stream);
  if (var == kVarGuard) return dispatch_ex2_subset<D, QG, KS, DUMP, kVarGuard>(kp, ex2, stream);
  if (var == kVarCausal) return dispatch_ex2_subset<D, QG, KS, DUMP, kVarCausal>(kp, ex2, stream);
  switch (ex2) {
    case 0: return launch_directp<D, QG, KS, DUMP, 0, kVarOnline>(kp, stream);
    case 1: return launch_directp<D, QG, KS, DUMP, 1, kVarOnline>(kp, stream);
    case 2: return launch_directp<D, QG, KS, DUMP, 2, kVarOnline>(kp, stream);
    case 4: return launch_directp<D, QG, KS, DUMP, 4, kVarOnline>(kp, stream);
    case 8: return launch_directp<D, QG, KS, DUMP, 8, kVarOnline>(kp, stream);
    case 16: return launch_directp<D, QG, KS, DUMP, 16, kVarOnline>(kp, stream);
    default: return hipErrorInvalidValue;
  }
}

template <int D, int QG, int KS>
hipError_t dispatch_dump(const KParams& kp, bool dump, int ex2, int var, hipStream_t stream) {
  return dump ? dispatch_ex2<D, QG, KS, true>(kp, ex2, var, stream) : dispatch_ex2<D, QG, KS, false>(kp, ex2, var, stream);
}

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
// / 19.3.  FP8 P/V with d = 128 leaves one wave per SIMD to four-wave workgroups (LDS):
// N 4096 U 128 52.6 / 65.9 / 38.8 / 26.3, U 256 54.5 / 67.0 / 42.8 / 48.0.
Shape choose_shape(int d, int N, int bh, bool causal, bool fp8) {
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
    // N that 256 does not divide (N 3968 U 744 110.9 against narrow's 148.0).
    if (W == 0 || (causal ? U <= 512 : W > 256 && W <= 384)) return half;
    return W > 128 ? wide : narrow;
  }
  if (fp8) {
    // d = 64: narrow workgroups, two per CU, throughout (N 4096 U 768 81.1 against wide's
    // 106.6, U 4096 376 / 418).
    return causal && U <= 512 && U <= N / 8 ? half : narrow;
  }
  if (d == 64) {
    // Four waves per SIMD (one-step pipeline).  Wide workgroups, two per CU, for whole
    // half rounds (+4-8 % on large shapes; -6 to -15 % where the last is partly
    // filled) and, causal, from 3072 of them (+2.5-5.7 %; -1 to -2 % at 1024-2048).
    if (causal ? U <= 640 && U <= N / 4 : U <= 512 && N >= 2048) return half;
    return W >= (causal ? 3072 : 256) && W % 256 == 0 ? wide : narrow;
  }
  if (causal) {
    // Wide from a round and a half on for long rows (N 4096 U 1024 57.0 against 58.9,
    // U 4096 238 / 247; N 8192 U 1024 95.2 / 103.4), but not between two rounds and four
    // (N 4096 U 1280 78.4 / 71.9), and never for short rows (N 2048 U 512 28.4 / 23.4, U 4096
    // 175 / 172; N 1024 U 1024 33.3 / 30.7).
    if (U <= 512 && U <= N / 8) return half;
    return N >= 4096 && ((W >= 384 && W <= 512) || W >= 1024) ? wide : narrow;
  }
  // Wide when more than half the CUs get one (N 4096 U 384 43.1 against 46.4, U 448 44.7 /
  // 48.5; N 512 even), except where the grid takes two to five rounds and the last is
  // at most half full: narrow workgroups, two per CU, finish that tail sooner (N 4096
  // U 768 78.3 / 85.4; at ten rounds 2 % slower).
  const bool tail = W > 256 && W <= 5 * 256 && W % 256 != 0 && W % 256 <= 128;
  return W > (N >= 1024 ? 128 : 255) && !tail ? wide : narrow;
}

template <int D>
hipError_t dispatch_shape(const KParams& kp, Shape s, bool dump, int ex2, int var, hipStream_t stream) {
  if (s.ks == 2) return dispatch_dump<D, 4, 2>(kp, dump, ex2, var, stream);
  if (s.ks == 4) return dispatch_dump<D, 2, 4>(kp, dump, ex2, var, stream);
  if (s.ks == 8) return dispatch_dump<D, 1, 8>(kp, dump, ex2, var, stream);
  return s.qg == 8 ? dispatch_dump<D, 8, 1>(kp, dump, ex2, var, stream) : dispatch_dump<D, 4, 1>(kp, dump, ex2, var, stream);
}

}  // namespace
}  // namespace directp_detail

hipError_t launch_forward_mxfp4(const DirectPArgs& a, hipStream_t stream) {
  using namespace directp_detail;
  KParams kp{};
  kp.qc = a.q_codes;
  kp.qs = a.q_scales;
  kp.kc = a.k_codes;
  kp.ks = a.k_scales;
  kp.vc = a.vt_codes;
  kp.vs = a.vt_scales;
  kp.out = a.out;
  kp.N = a.N;
  // fp32 coefficients of the folded code map (see the file header).
  const double s = (double)a.softmax_scale, A = (double)a.affine_a, Bc = (double)a.affine_b;
  kp.c_y = (float)(s * kLog2E / 36.0);
  const float c_a = (float)(A * s * kLog2E / 36.0);
  const float k0 = (float)(A * kLog2Of6 + Bc);
  kp.c_a8 = c_a * 0.125f;
  kp.k0_8 = k0 * 0.125f;
  kp.a8 = a.affine_a * 0.125f;
  kp.k1 = (float)kLog2Of6;
  kp.margin = (float)a.guard_margin;
  kp.floor_u = (float)(a.guard_shift + 1);
  kp.shift = (float)a.guard_shift;
  kp.out_bf16 = a.out_bf16;
  kp.row_ids = a.row_ids;
  kp.n_rows = a.n_rows;
  kp.p_codes = a.p_codes;
  kp.block_exp = a.block_exp;
  kp.row_m = a.row_m;
  kp.row_d = a.row_d;
  kp.wg_clock = a.wg_clock;
  kp.lse = a.lse;
  const bool dump = a.n_rows > 0;
  const int bh = a.B * a.H;
  const int ex2 = a.ex2_pairs;
  const int var = (a.guard ? kVarGuard : (a.causal ? kVarCausal : kVarOnline)) | (a.pv_fp8 ? kPV8 : 0);
  const Shape shape = choose_shape(a.d, a.N, bh, a.causal != 0, a.pv_fp8 != 0);
  kp.n_qtiles = a.N / (32 * shape.qg);
  kp.total = kp.n_qtiles * bh;
  kp.n_clock = (int)((int64_t)bh * a.N / 128);
  return a.d == 128 ? dispatch_shape<128>(kp, shape, dump, ex2, var, stream)
                    : dispatch_shape<64>(kp, shape, dump, ex2, var, stream);
}

}  // namespace fp4attn
