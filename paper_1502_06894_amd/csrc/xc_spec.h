// Spectrum stores of the F stage: FP32 complex, or for the MFMA X path the
// power-of-two-scaled value as FP16 (Re, Im) or OCP e4m3 (Re, Im).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xc_launch.h"

namespace xc {

// NT: non-temporal stores, for a wave that writes whole lines (consecutive
// channels): a block's spectra (gigabytes) are read back by the X stage only
// after the whole block is written, so keeping them in the caches would only
// evict lines that are still useful (measured on MI355X: the X stage that
// follows runs 9 % faster).  Scattered stores (every 16th channel, the
// N = 32768 row kernel) stay ordinary so that the cache merges their lines.
template <typename V>
__device__ inline void store_spec(V* p, V v, bool nt) {
  if (nt)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <int OUT, bool NT = true>
__device__ inline void put_spec(void* spec, size_t idx, float2 y, int e) {
  if constexpr (OUT == kOutF32) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {y.x, y.y};
    store_spec(static_cast<f2*>(spec) + idx, v, NT);
  } else if constexpr (OUT == kOutF16) {
    const float sx = ldexpf(y.x, e), sy = ldexpf(y.y, e);
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    h2 h;
    h.x = (_Float16)sx;
    h.y = (_Float16)sy;
    store_spec(static_cast<h2*>(spec) + idx, h, NT);
  } else {
    // the conversion maps overflow to NaN: saturate at the e4m3 maximum first
    const float sx = fminf(fmaxf(ldexpf(y.x, e), -448.f), 448.f);
    const float sy = fminf(fmaxf(ldexpf(y.y, e), -448.f), 448.f);
    const int pk = __builtin_amdgcn_cvt_pk_fp8_f32(sx, sy, 0, false);
    store_spec(static_cast<uint16_t*>(spec) + idx, (uint16_t)(pk & 0xffff), NT);
  }
}

}  // namespace xc
