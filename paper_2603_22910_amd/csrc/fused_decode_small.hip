// Kernel instantiations of fused_decode_small.h (a translation unit of its own: they take as long to
// compile as the rest of the library).
#include "fused_decode_small.h"

namespace echokv {

template <typename T, int HD, int TB>
static int launch(const fsmall::Args<T>& a, const StreamMeta& mt, bool packed, hipStream_t st) {
  const dim3 g(a.n_fused + a.streams.n_ret + a.streams.n_win), blk(fsmall::NTHREADS);
  const bool rope = a.rope_cos != nullptr;
#define ECHOKV_SMALL_CASE(PK_) \
  do { if (rope) hipLaunchKernelGGL((fsmall::fused_decode_small_kernel<T, HD, TB, PK_, true>), g, blk, 0, st, a, mt); \
       else hipLaunchKernelGGL((fsmall::fused_decode_small_kernel<T, HD, TB, PK_, false>), g, blk, 0, st, a, mt); } while (0)
  if constexpr (sizeof(T) == 2) { if (packed) ECHOKV_SMALL_CASE(true); else ECHOKV_SMALL_CASE(false); }
  else ECHOKV_SMALL_CASE(false);
#undef ECHOKV_SMALL_CASE
  return hipGetLastError() != hipSuccess ? 7 : 0;
}

template <typename T>
int launch_fused_decode_small(const fsmall::Args<T>& a, const StreamMeta& mt, int tb, bool packed, hipStream_t st) {
  constexpr int LO = sizeof(T) == 2 ? 2 : 1, HI = 2 * LO;
  if (tb != LO && tb != HI) return 2;
  if (a.streams.ret.d == 128) return tb == LO ? launch<T, 128, LO>(a, mt, packed, st) : launch<T, 128, HI>(a, mt, packed, st);
  return tb == LO ? launch<T, 64, LO>(a, mt, packed, st) : launch<T, 64, HI>(a, mt, packed, st);
}
template int launch_fused_decode_small<bf16_t>(const fsmall::Args<bf16_t>&, const StreamMeta&, int, bool, hipStream_t);
template int launch_fused_decode_small<float>(const fsmall::Args<float>&, const StreamMeta&, int, bool, hipStream_t);

}  // namespace echokv
