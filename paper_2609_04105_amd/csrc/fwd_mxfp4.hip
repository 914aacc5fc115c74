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
  const Shape shape = directp_shape(a.d, a.N, bh, a.causal != 0, a.pv_fp8 != 0);
  kp.n_qtiles = a.N / (32 * shape.qg);
  kp.total = kp.n_qtiles * bh;
  kp.n_clock = (int)((int64_t)bh * a.N / 128);
  return a.d == 128 ? dispatch_shape<128>(kp, shape, dump, ex2, var, stream)
                    : dispatch_shape<64>(kp, shape, dump, ex2, var, stream);
}

}  // namespace fp4attn
