// Host side of the decayed-load scoring (online_kernel.h), and its launches for top_k > 8.
#include "online_kernel.h"

namespace tacg {
namespace {

__global__ __launch_bounds__(256) void on_zero(OnArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t j = i; j < a.P; j += stride) {
    a.cost_home[j] = 0;
    a.cost_span[j] = 0;
  }
  if (a.cost_home_fam)
    for (int64_t j = i; j < static_cast<int64_t>(a.P) * a.F; j += stride) a.cost_home_fam[j] = 0;
}

}  // namespace

int launch_eval_online(const int16_t* trace, int64_t N, int32_t L, int32_t K, int32_t E, const int64_t* fam_off_host,
                       int32_t F, const int32_t* home_start_host, const int32_t* home_size_host, int32_t G, int32_t P,
                       const uint8_t* primary, const uint8_t* secondary, int32_t R, double rho, int32_t theta_num,
                       int32_t theta_den, const double* state_in, double* state_out, uint64_t* cost_home,
                       uint64_t* cost_span, uint32_t* load, uint64_t* cost_home_fam, uint32_t* d_err,
                       hipStream_t stream) {
  OnArgs a{};
  a.trace = trace;
  a.primary = primary;
  a.secondary = R > 0 ? secondary : nullptr;
  a.state_in = state_in;
  a.state_out = state_out;
  a.cost_home = reinterpret_cast<unsigned long long*>(cost_home);
  a.cost_span = reinterpret_cast<unsigned long long*>(cost_span);
  a.load = load;
  a.cost_home_fam = reinterpret_cast<unsigned long long*>(cost_home_fam);
  a.d_err = d_err;
  a.rho = rho;
  a.N = N;
  a.L = L;
  a.K = K;
  a.E = E;
  a.F = F;
  a.G = G;
  a.P = P;
  a.R = R;
  a.theta_num = theta_num;
  a.theta_den = theta_den;
  for (int f = 0; f < F; ++f)
    a.fam[f] = make_uint4(static_cast<uint32_t>(fam_off_host[f]), static_cast<uint32_t>(fam_off_host[f + 1]),
                          static_cast<uint32_t>(home_start_host[f]) |
                              (static_cast<uint32_t>(home_size_host[f]) << 8),
                          0u);
  // sentinel past the last family: a token index never reaches its end
  for (int f = F; f < TACG_MAX_FAMILIES; ++f) a.fam[f] = make_uint4(0xffffffffu, 0xffffffffu, 1u << 8, 0u);
  hipLaunchKernelGGL(on_zero, dim3(64), dim3(256), 0, stream, a);
  if (P > 0) {
    switch (K) {
#define TACG_K(k)              \
  case k:                      \
    launch_on<k>(a, stream);   \
    break;
      case 1: case 2: case 3: case 4: case 5: case 6: case 7: case 8:
        launch_online_low(a, stream);
        break;
      TACG_K(9) TACG_K(10) TACG_K(11) TACG_K(12) TACG_K(13) TACG_K(14) TACG_K(15) TACG_K(16)
#undef TACG_K
      default:
        return TACG_E_UNSUPPORTED;
    }
  }
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

}  // namespace tacg
