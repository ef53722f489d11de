// Launches of the decayed-load scoring for top_k <= 8 (a translation unit of its own: the kernels of one take a minute and a
// half to compile).
#include "online_kernel.h"

namespace tacg {

void launch_online_low(const OnArgs& a, hipStream_t stream) {
  switch (a.K) {
#define TACG_K(k)              \
  case k:                      \
    launch_on<k>(a, stream);   \
    break;
    TACG_K(1) TACG_K(2) TACG_K(3) TACG_K(4) TACG_K(5) TACG_K(6) TACG_K(7) TACG_K(8)
#undef TACG_K
    default:
      break;
  }
}

}  // namespace tacg
