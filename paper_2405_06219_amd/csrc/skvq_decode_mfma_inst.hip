// One (K format, V format) pair of the matrix-core decode kernels: compiled once per pair with
// -DSKVQ_KL=<key levels> -DSKVQ_VL=<value levels> (the pairs are listed in build.py and in the
// dispatcher, skvq_decode_mfma.hip).
#include "skvq_decode_mfma_kernel.h"
#include "skvq_decode_wide_kernel.h"

#if !defined(SKVQ_KL) || !defined(SKVQ_VL)
#error "compile with -DSKVQ_KL=4|8|16 -DSKVQ_VL=3|4|8|16"
#endif

namespace skvq {

// The launcher of the kernels with KL-level keys and VL-level values.
template <int KL, int VL>
hipError_t launch_decode_mfma_fmt(const Layout &L, const __half *q, long long T, long long nq, int n_sink,
                                  DecodePlan shape, int n_new, const __half *knew, const __half *vnew, long long te,
                                  MergeOut mo, hipStream_t s) {
  const int n_splits = shape.n_splits, passes = shape.passes;
  if (T <= 0 || nq < 0 || nq > SKVQ_MAX_QUANT_TOKENS || T - nq > 0x7fffffff || n_splits < 1 ||
      n_splits > SKVQ_MAX_SPLITS)
    return hipErrorInvalidValue;
  if (n_new < 1 || n_new > SKVQ_MAX_NEW_TOKENS || L.R > 8) return hipErrorInvalidValue;
  const int n_rows = n_new * L.R;
  const bool wide = shape.rows == kWideRows;
  if ((!wide && shape.rows != kNarrowRows) || passes != decode_passes(n_rows, shape.rows)) return hipErrorInvalidValue;
  if (wide && (L.NG > 2 || L.uneq)) return hipErrorInvalidValue;
  const int rk = wide ? kWideRows : n_rows == 1 ? 1 : n_rows == 2 ? 2 : kNarrowRows;
  if ((knew != nullptr) != (vnew != nullptr) || (knew && (passes != 1 || n_new != 1))) return hipErrorInvalidValue;
  if (knew && T - 1 >= L.W && (te < 0 || te >= L.Tcap || te != nq - 1)) return hipErrorInvalidValue;
  if ((long long)L.Hk * passes > 65535) return hipErrorInvalidValue;
  if (mo.mode != kMergeSeparate && !mo.out_f32) return hipErrorInvalidValue;
  if (mo.mode == kMergeDirect && n_splits != 1) return hipErrorInvalidValue;
  const dim3 grid(n_splits, L.Hk * passes, L.B), block(kThreads);
  const ChunkPlan plan = plan_chunks(L, T, nq, n_sink, n_splits, knew != nullptr, !wide && knew != nullptr && te >= 0);
#define SKVQ_LAUNCH(RR, MM, GG, UU)                                                                                  \
  hipLaunchKernelGGL((decode_mfma_kernel<RR, KL, VL, MM, GG, UU>), grid, block, 0, s, L, q, T, nq, n_sink, n_splits, \
                     passes, n_new, knew, vnew, te, plan, mo)
#define SKVQ_LAUNCH_WIDE(MM, GG)                                                                             \
  hipLaunchKernelGGL((decode_wide_kernel<KL, VL, MM, GG>), grid, block, 0, s, L, q, T, nq, n_sink, n_splits, \
                     passes, n_new, knew, vnew, te, plan, mo)
#define SKVQ_LAUNCH_NG(RR, MM)                                                                   \
  switch (L.NG) {                                                                                \
    case 1: SKVQ_LAUNCH(RR, MM, 1, false); break;                                                \
    case 2: if (L.uneq) SKVQ_LAUNCH(RR, MM, 2, true); else SKVQ_LAUNCH(RR, MM, 2, false); break; \
    case 4: if (L.uneq) SKVQ_LAUNCH(RR, MM, 4, true); else SKVQ_LAUNCH(RR, MM, 4, false); break; \
    default: return hipErrorInvalidValue;                                                        \
  }
#define SKVQ_LAUNCH_META(RR)                                                \
  switch (L.meta_fmt) {                                                     \
    case SKVQ_META_F32: SKVQ_LAUNCH_NG(RR, SKVQ_META_F32) break;            \
    case SKVQ_META_F16: SKVQ_LAUNCH_NG(RR, SKVQ_META_F16) break;            \
    case SKVQ_META_FP8_E4M3: SKVQ_LAUNCH_NG(RR, SKVQ_META_FP8_E4M3) break;  \
    default: return hipErrorInvalidValue;                                   \
  }
  if (L.k_levels != KL || L.v_levels != VL) return hipErrorInvalidValue;
  switch (rk) {
    case 1: SKVQ_LAUNCH_META(1) break;
    case 2: SKVQ_LAUNCH_META(2) break;
    case 4: SKVQ_LAUNCH_META(4) break;
    case kWideRows:
      switch (L.meta_fmt) {
        case SKVQ_META_F32: if (L.NG == 1) SKVQ_LAUNCH_WIDE(SKVQ_META_F32, 1); else SKVQ_LAUNCH_WIDE(SKVQ_META_F32, 2); break;
        case SKVQ_META_F16: if (L.NG == 1) SKVQ_LAUNCH_WIDE(SKVQ_META_F16, 1); else SKVQ_LAUNCH_WIDE(SKVQ_META_F16, 2); break;
        case SKVQ_META_FP8_E4M3:
          if (L.NG == 1) SKVQ_LAUNCH_WIDE(SKVQ_META_FP8_E4M3, 1); else SKVQ_LAUNCH_WIDE(SKVQ_META_FP8_E4M3, 2);
          break;
        default: return hipErrorInvalidValue;
      }
      break;
    default: return hipErrorInvalidValue;
  }
#undef SKVQ_LAUNCH_META
#undef SKVQ_LAUNCH_NG
#undef SKVQ_LAUNCH
#undef SKVQ_LAUNCH_WIDE
  return hipGetLastError();
}

template hipError_t launch_decode_mfma_fmt<SKVQ_KL, SKVQ_VL>(const Layout &, const __half *, long long, long long,
                                                             int, DecodePlan, int, const __half *, const __half *, long long,
                                                             MergeOut, hipStream_t);
}  // namespace skvq
