// Grouping objective of Sec. 3.3 (eq. grouping-objective) for many placements: the within-group
// affinity  obj[p][l] = sum_m sum_{e != e' on GPU m} A-tilde_l(e, e'),  accumulated in float64.
//
// group_objective_kernel (many placements): lane = placement; a workgroup takes SETS x 64 placements of one layer, SETS of
// them per lane.
//   1. One wave per 64 placements links the experts of every GPU into a ring, next[e][lane][set] in LDS: going
//      down the expert ids, one LDS exchange of the GPU's head with the expert yields its successor; the
//      last expert of a GPU is linked to its first at the end.  Heads and tails are lane-private dwords, and the
//      four set bytes of a lane share a dword, so a lane always reads its own LDS bank.
//   2. The waves share the experts.  For its expert e a wave stages row e of A-tilde in its own KB of LDS, and every
//      lane walks its placement's ring of e's GPU, adding the row's entries: two LDS reads and one float64
//      add per pair, all lanes busy when the GPUs hold equally many experts.
//   3. The waves' sums are added in wave order.
// What bounds it, by counters: the latency of an entry's two dependent LDS reads (the waves wait 62 % of their time; VALU 45 % busy,
// bank conflicts of the random row entries 14 % of the time).  Measured on MI355X at E = 256, 32 GPUs, 1024
// placements x 58 layers (1.1e8 entries), device time: 427 -> 67 us against one workgroup per (placement, layer).
//
// group_gather_kernel (few placements): one workgroup per (placement, layer) lists the experts of every GPU by ballots, then
// thread e gathers the entries of its own A-tilde row at the other members of its GPU from L2.  Bound by the cache
// lines per load once the chip is full; below that its chain is one GPU's members long, where a wave of the rings walks
// E / 16 of them (the rings take about as long for one placement as for 64).
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

// Few placements.  grid (P, L), one thread per expert.
constexpr int kGatherThreads = 256;

__global__ __launch_bounds__(kGatherThreads) void group_gather_kernel(const float* __restrict__ a_tilde, int L, int E,
                                                                      const uint8_t* __restrict__ primary, int G,
                                                                      double* __restrict__ obj, uint32_t* d_err) {
  constexpr int kGatherWaves = kGatherThreads / 64;
  __shared__ unsigned long long lanes_of[kGatherWaves][TACG_MAX_GPUS];  // lanes of each wave holding GPU m
  __shared__ int start[TACG_MAX_GPUS + 1];                              // list offsets per GPU
  __shared__ uint8_t member[TACG_MAX_EXPERTS];                          // experts grouped by GPU, ids increasing
  __shared__ double part[kGatherWaves];
  const int p = blockIdx.x, l = blockIdx.y;
  const int e = threadIdx.x;
  const int lane = e & 63, wave = e >> 6;
  uint32_t err = 0;
  uint32_t g = 0xFF;  // 0xFF: no expert, or left out of every group (a table error)
  if (e < E) {
    g = primary[(static_cast<int64_t>(p) * L + l) * E + e];
    if (g >= static_cast<uint32_t>(G)) {
      err = TACG_ERR_TABLE;
      g = 0xFF;
    }
  }
  for (int m = 0; m < G; ++m) {
    const unsigned long long b = __ballot(g == static_cast<uint32_t>(m));
    if (lane == 0) lanes_of[wave][m] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0;
    for (int m = 0; m < G; ++m) {
      start[m] = s;
      for (int w = 0; w < kGatherWaves; ++w) s += __popcll(lanes_of[w][m]);
    }
    start[G] = s;
  }
  __syncthreads();
  if (g != 0xFF) {
    int rank = __popcll(lanes_of[wave][g] & ((1ull << lane) - 1ull));
    for (int w = 0; w < wave; ++w) rank += __popcll(lanes_of[w][g]);
    member[start[g] + rank] = static_cast<uint8_t>(e);
  }
  __syncthreads();
  double acc = 0.0;
  if (g != 0xFF) {
    const float* row = a_tilde + (static_cast<int64_t>(l) * E + e) * E;
    const int b0 = start[g], b1 = start[g + 1];
#pragma unroll 4
    for (int i = b0; i < b1; ++i) {
      const int e2 = member[i];
      if (e2 != e) acc += static_cast<double>(row[e2]);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) part[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kGatherWaves; ++w) s += part[w];
    obj[static_cast<int64_t>(p) * L + l] = s;
  }
  if (err) atomicOr(d_err, err);
}

// Where the gather takes over: placements x layers, by the experts per GPU (its time grows with all three, the rings' only
// with the last until their workgroups fill the chip).  Device times on MI355X, gather / rings in us, 12 layers: 256 experts on
// one GPU 287 / 305 at 1080 rows, 415 / 304 at 1560; on 4 109 / 97 at 1560; on 8 56 / 62 at 1560, 67 / 62 at 2040; on 16 45 / 45 at
// 2580; on 32 33 / 38 at 3600, 41 / 39 at 4800 (58 layers: 35 / 39 at 3016); 128 on 2 50 / 50 at 1508; on 16 17 / 20 at 3072, 22 / 20
// at 4800; 64 on 32 9.4 / 11.6 at 2040, 12.0 / 11.7 at 2580; 33 on one 9.0 / 11.2 at 2040, 13.3 / 11.1 at 2580; 16 on 4 4.7 /
// 5.0 at 2040, 6.1 / 4.7 at 2580.  One placement of 2 layers: 256 experts on 2, 8 and 32 GPUs 25 / 180, 11 / 74 and 9 / 44.
bool group_uses_gather(int64_t rows, int E, int G) {
  int64_t limit = 2432;                 // fewer than four experts per GPU
  if (E < 32) limit = 2048;
  else if (E < 40 && E > 8 * G) limit = 2240;
  else if (E > 64 * G) limit = 1152;
  else if (E > 32 * G) limit = 1408;
  else if (E > 16 * G) limit = 1856;
  else if (E > 8 * G) limit = 2560;
  else if (E >= 4 * G) limit = 3456;
  return rows <= limit;
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
  if (group_uses_gather(static_cast<int64_t>(P) * L, E, G)) {
    hipLaunchKernelGGL(group_gather_kernel, dim3(P, L), dim3(kGatherThreads), 0, stream, a_tilde, L, E, primary, G, obj, d_err);
    return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
  }
  // as many placements per workgroup as still leave the chip about one workgroup per CU (a workgroup's rows of A-tilde
  // serve all its placements); 192 is three quarters of the CUs, chosen and not swept
  const int64_t sets = (P + 63) / 64;
  if ((sets + 3) / 4 * L >= 192) launch_sets<4>(a_tilde, L, E, primary, P, G, obj, d_err, stream);
  else if ((sets + 1) / 2 * L >= 192) launch_sets<2>(a_tilde, L, E, primary, P, G, obj, d_err, stream);
  else launch_sets<1>(a_tilde, L, E, primary, P, G, obj, d_err, stream);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

}  // namespace tacg
