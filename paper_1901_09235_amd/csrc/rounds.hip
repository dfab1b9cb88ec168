// rounds.hip -- the round kernel's instances of one type (DCDL_R) and workgroup
// size (DCDL_NT); the build compiles this file once for each.
#include "dcdl_device.h"

namespace dcdl {

template <bool EXT> static const void *rounds_kernel_ng(int ng) {
  switch (ng) {
    case 1: return reinterpret_cast<const void *>(lgcd_rounds<DCDL_R, DCDL_NT, 1, EXT>);
    case 2: return reinterpret_cast<const void *>(lgcd_rounds<DCDL_R, DCDL_NT, 2, EXT>);
    case 3: return reinterpret_cast<const void *>(lgcd_rounds<DCDL_R, DCDL_NT, 3, EXT>);
    default: return reinterpret_cast<const void *>(lgcd_rounds<DCDL_R, DCDL_NT, 0, EXT>);
  }
}

template <> const void *rounds_kernel<DCDL_R, DCDL_NT>(int ng, bool ext) {
  return ext ? rounds_kernel_ng<true>(ng) : rounds_kernel_ng<false>(ng);
}

}  // namespace dcdl
