// Launcher of the segmented family for ONE storage type: this file is compiled
// once per storage type (-DHDC_SEG_STORAGE=F32|F16|BF16|I32 with the matching
// -DHDC_SEG_NAME=run_segmented_f32|...), as the fused map + reduce family is.
#include "hdc_launch.hpp"

#if !defined(HDC_SEG_STORAGE) || !defined(HDC_SEG_NAME)
#error "define HDC_SEG_STORAGE and HDC_SEG_NAME"
#endif

namespace hdc {

hdc_status HDC_SEG_NAME(const hdc_functor& f, const void* x, const int64_t* off, int64_t nseg, int64_t total,
                        hdc_accum acc, void* out, void* ws, size_t ws_bytes, uint32_t* ticket, const Tuning& t,
                        hipStream_t st) {
  using S = HDC_SEG_STORAGE;
  if constexpr (std::is_same_v<S, I32>) {
    (void)acc;
    return with_int_fn(f, [&](auto fn) {
      return launch_segmented<decltype(fn), I32, IntAcc>(fn, x, off, nseg, total, out, ws, ws_bytes, ticket, t, st);
    });
  } else {
    return with_float_fn(f, [&](auto fn) -> hdc_status {
      using F = decltype(fn);
      if constexpr (F::binary) {
        return fail(HDC_ERR_UNSUPPORTED, "PRODUCT is not a segmented fold term");
      } else {
        if (acc == HDC_ACC_COMPENSATED)
          return launch_segmented<F, S, CompAcc>(fn, x, off, nseg, total, out, ws, ws_bytes, ticket, t, st);
        return launch_segmented<F, S, PlainAcc>(fn, x, off, nseg, total, out, ws, ws_bytes, ticket, t, st);
      }
    });
  }
}

}  // namespace hdc
