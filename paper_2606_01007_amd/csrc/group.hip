// Grouping objective of Sec. 3.3 (eq. grouping-objective) for many placements: the within-group
// affinity  obj[p][l] = sum_m sum_{e != e' on GPU m} A-tilde_l(e, e'),  accumulated in float64.
//
// Lane = placement; a workgroup takes SETS x 64 placements of one layer, SETS of them per lane.
//   1. One wave per 64 placements links the experts of every GPU into a ring, next[e][lane][set] in LDS: going
//      down the expert ids, one LDS exchange of the GPU's head with the expert yields its successor; the
//      last expert of a GPU is linked to its first at the end.  Heads and tails are lane-private dwords, and the
//      four set bytes of a lane share a dword, so a lane always reads its own LDS bank.
//   2. The waves share the experts.  For its expert e a wave stages row e of A-tilde in its own KB of LDS, and every
//      lane walks its placement's ring of e's GPU, adding the row's entries: two LDS reads and one float64
//      add per pair, all lanes busy when the GPUs hold equally many experts.
//   3. The waves' sums are added in wave order.
//
// What bounds it: the row entries' LDS reads (random banks) and VALU issue.  Gathering the
// entries from L2 instead, one lane per expert with lists by ballots, was bound by the cache lines per load.
// Measured on MI355X at E = 256, 32 GPUs, 1024 placements x 58 layers (1.1e8 entries): 427 -> 67 us.
#include "tacg_internal.h"

namespace tacg {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kRingRow = 256;   // bytes of next[e]: 64 lanes x 4 sets
constexpr int kLink = 16;       // experts linked at once
constexpr uint32_t kNoExpert = 0xffffffffu;

// LDS: head [G + 1][64] and tail [G + 1][64] dwords per set, rings [E][kRingRow], rows [kWaves][E] floats; the sums
// [kWaves][64] float64 per set go over the heads, tails and rings, which are free by then
__host__ __device__ inline size_t row_off(int sets, int E, int G) {
  const size_t lists = static_cast<size_t>(sets) * 2 * (G + 1) * 64 * 4 + static_cast<size_t>(E) * kRingRow;
  const size_t sums = static_cast<size_t>(sets) * kWaves * 64 * 8;
  return lists > sums ? lists : sums;
}

template <bool WORDS, int kSets>  // WORDS: the placement rows are dword-aligned
__global__ __launch_bounds__(kThreads) void group_objective_kernel(const float* __restrict__ a_tilde, int L, int E,
                                                                   const uint8_t* __restrict__ primary, int P, int G,
                                                                   double* __restrict__ obj, uint32_t* d_err) {
  extern __shared__ __align__(16) char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = blockIdx.y, p0 = blockIdx.x * (64 * kSets);
  char* const rings = lds + static_cast<size_t>(kSets) * 2 * (G + 1) * 64 * 4;
  uint32_t err = 0;

  // ---- the rings ----
  if (wave < kSets) {
    // row G of the heads and tails takes the experts left out by a table error and the writes not wanted
    uint32_t* const head = reinterpret_cast<uint32_t*>(lds) + wave * 2 * (G + 1) * 64 + lane;
    uint32_t* const tail = head + (G + 1) * 64;
    char* const next = rings + lane * 4 + wave;
    const int p = p0 + wave * 64 + lane;
    const bool live = p < P;
    const uint8_t* src = primary + (static_cast<int64_t>(min(p, P - 1)) * L + l) * E;
    for (int g = 0; g <= G; ++g) head[g * 64] = kNoExpert;
    // kLink experts at once, from the highest id down: their exchanges are all in flight before the first result is used
    auto link = [&](int e0, const uint32_t (&gpu)[kLink]) {
      uint32_t g[kLink], after[kLink];
#pragma unroll
      for (int i = kLink - 1; i >= 0; --i) {
        const bool ok = gpu[i] < static_cast<uint32_t>(G);
        err |= (live && !ok && e0 + i >= 0) ? TACG_ERR_TABLE : 0u;
        g[i] = ok && e0 + i >= 0 ? gpu[i] : static_cast<uint32_t>(G);
        after[i] = __hip_atomic_exchange(head + g[i] * 64, static_cast<uint32_t>(e0 + i), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
      }
#pragma unroll
      for (int i = kLink - 1; i >= 0; --i) {
        if (e0 + i < 0) continue;
        const uint32_t e = static_cast<uint32_t>(e0 + i);
        const bool out = g[i] == static_cast<uint32_t>(G);
        next[e * kRingRow] = static_cast<char>(out ? e : after[i]);
        tail[(after[i] == kNoExpert ? g[i] : static_cast<uint32_t>(G)) * 64] = e;
      }
    };
    constexpr int kWords = kLink / 4;
    uint32_t ahead[WORDS ? kWords : kLink];  // the next step's GPUs are in flight while one is linked
    auto fetch = [&](int e0) {
      if constexpr (WORDS) {  // E is a multiple of four, and so is e0
#pragma unroll
        for (int i = 0; i < kWords; ++i) ahead[i] = reinterpret_cast<const uint32_t*>(src)[max(e0 / 4 + i, 0)];
      } else {
#pragma unroll
        for (int i = 0; i < kLink; ++i) ahead[i] = src[max(e0 + i, 0)];
      }
    };
    fetch(E - kLink);
    for (int e0 = E - kLink; e0 > -kLink; e0 -= kLink) {
      uint32_t gpu[kLink];
#pragma unroll
      for (int i = 0; i < kLink; ++i) gpu[i] = WORDS ? (ahead[i / 4] >> (8 * (i & 3))) & 0xffu : ahead[WORDS ? 0 : i];
      fetch(e0 - kLink);
      link(e0, gpu);
    }
    for (int g = 0; g < G; ++g) {
      const uint32_t hd = head[g * 64];
      if (hd != kNoExpert) next[tail[g * 64] * kRingRow] = static_cast<char>(hd);
    }
  }
  barrier_after_lds_atomics();

  // ---- the pairs: expert by expert, every placement's ring ----
  float* const row = reinterpret_cast<float*>(lds + row_off(kSets, E, G)) + wave * E;
  const float* const al = a_tilde + static_cast<int64_t>(l) * E * E;
  double acc[kSets] = {};
  float ahead[4];
  auto fetch = [&](int e) {
    const float* src = al + static_cast<int64_t>(min(e, E - 1)) * E;
#pragma unroll
    for (int q = 0; q < 4; ++q) ahead[q] = src[min(lane + 64 * q, E - 1)];
  };
  fetch(wave);
  for (int e = wave; e < E; e += kWaves) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (lane + 64 * q < E) row[lane + 64 * q] = lane + 64 * q == e ? 0.0f : ahead[q];
    fetch(e + kWaves);
    __asm__ __volatile__("" ::: "memory");  // the LDS keeps a wave's operations in order
    uint32_t at[kSets];
    const uint8_t* const nx = reinterpret_cast<const uint8_t*>(rings) + lane * 4;
#pragma unroll
    for (int s = 0; s < kSets; ++s) at[s] = nx[e * kRingRow + s];
    const uint32_t ue = static_cast<uint32_t>(e);
    // a lane whose ring is done stays on e, whose entry counts as zero; every ring closes within E steps
    for (int step = 0; step < E; step += 2) {
      bool more = false;
#pragma unroll
      for (int s = 0; s < kSets; ++s) more |= at[s] != ue;
      if (!__any(more)) break;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int s = 0; s < kSets; ++s) {
          const float x = row[at[s]];
          const uint32_t to = nx[at[s] * kRingRow + s];
          acc[s] += static_cast<double>(x);
          at[s] = at[s] != ue ? to : ue;
        }
      }
    }
    __asm__ __volatile__("" ::: "memory");
  }
  __syncthreads();  // every wave is done with the rings
  double* const sums = reinterpret_cast<double*>(lds);  // [kSets][kWaves][64]
#pragma unroll
  for (int s = 0; s < kSets; ++s) sums[(s * kWaves + wave) * 64 + lane] = acc[s];
  __syncthreads();
  if (wave < kSets) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += sums[(wave * kWaves + w) * 64 + lane];
    const int p = p0 + wave * 64 + lane;
    if (p < P) obj[static_cast<int64_t>(p) * L + l] = t;
  }
  if (err) atomicOr(d_err, err);
}

template <int kSets>
void launch_sets(const float* a_tilde, int L, int E, const uint8_t* primary, int P, int G, double* obj, uint32_t* d_err,
                 hipStream_t stream) {
  const size_t lds = row_off(kSets, E, G) + static_cast<size_t>(kWaves) * E * sizeof(float);
  const dim3 grid((P + 64 * kSets - 1) / (64 * kSets), L);
  const bool words = E % 4 == 0 && reinterpret_cast<uintptr_t>(primary) % 4 == 0;
  auto* kernel = words ? &group_objective_kernel<true, kSets> : &group_objective_kernel<false, kSets>;
  allow_lds(kernel, lds);
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), lds, stream, a_tilde, L, E, primary, P, G, obj, d_err);
}

}  // namespace

int launch_group_objective(const float* a_tilde, int32_t L, int32_t E, const uint8_t* primary, int32_t P, int32_t G,
                           double* obj, uint32_t* d_err, hipStream_t stream) {
  // as many placements per workgroup as still leave the chip about one workgroup per CU (a workgroup's rows of A-tilde
  // serve all its placements)
  const int64_t sets = (P + 63) / 64;
  if ((sets + 3) / 4 * L >= 192) launch_sets<4>(a_tilde, L, E, primary, P, G, obj, d_err, stream);
  else if ((sets + 1) / 2 * L >= 192) launch_sets<2>(a_tilde, L, E, primary, P, G, obj, d_err, stream);
  else launch_sets<1>(a_tilde, L, E, primary, P, G, obj, d_err, stream);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

}  // namespace tacg
