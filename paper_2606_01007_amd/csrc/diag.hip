// Motivation diagnostics of App. H (auxiliary metrics) from the co-activation counts:
//   * activation Frobenius distance between the expert-activation distributions of two families,
//     P_f[l][e] = D_f[l][e] / N_{f,l}, dist[i][j] = ||P_i - P_j||_F over all layers and experts;
//   * top-n co-activated pair sets per (family, layer) and their Jaccard overlaps per layer.
//
// dist_kernel: one workgroup per unordered family pair, one wave per layer (wave sums only), float64.
// top_pairs_kernel: one workgroup per (family, layer).  The segment's upper triangle is read once, into registers:
//   rows a and E - 1 - a together hold E - 1 pairs, so a wave takes such row pairs, four dwords per lane each.  The
//   n-th largest positive count T is found by bisection in one wave, first over the threads' maxima (a lower
//   bound), then over the list of the counts at or above that bound; pairs above T are kept, ties at T in increasing pair order until n are chosen: the rows' counts of
//   both are prefix-summed, which gives every row its ties to keep and its first output slot, and
//   ballots give the order within a row.  Bound, by counters, by latency, that of the triangle's read (rows of C) and of
//   the steps between barriers (the waves wait 77 % of their time; VALU 21 % busy); two workgroups per CU.  Measured on MI355X at E = 256, 16 families, 58 layers, n = 64:
//   277 -> 73 us (the triangle staged in 130 KB of LDS and scanned there, one workgroup per CU).
// jaccard_kernel: one wave per (layer, unordered family pair); every element of one sorted list is looked up
//   in the other by bisection.
#include <algorithm>

#include "tacg_internal.h"

namespace tacg {
namespace {

constexpr int kDistThreads = 1024;
constexpr int kTopThreads = 1024;

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__global__ __launch_bounds__(kDistThreads) void dist_kernel(const uint32_t* __restrict__ D, int F, int L, int E, int k,
                                                            double* __restrict__ dist) {
  __shared__ double dred[kDistThreads / 64];
  const int i = blockIdx.x, j = blockIdx.y;
  if (i > j) return;  // the distance of (j, i) is written with that of (i, j)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  double acc = 0.0;
  for (int l = wave; l < L; l += nw) {  // one wave per layer, lanes over experts
    const uint32_t* Di = D + (static_cast<int64_t>(i) * L + l) * E;
    const uint32_t* Dj = D + (static_cast<int64_t>(j) * L + l) * E;
    uint32_t di[4], dj[4];
    unsigned long long si = 0, sj = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = lane + 64 * q;
      di[q] = e < E ? Di[e] : 0u;
      dj[q] = e < E ? Dj[e] : 0u;
      si += di[q];
      sj += dj[q];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      si += __shfl_xor(si, o, 64);
      sj += __shfl_xor(sj, o, 64);
    }
    // P = D / N with N = sum_e D / k, i.e. P = k * D / sum_e D (0 for an empty family)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double pi = si ? static_cast<double>(di[q]) / (static_cast<double>(si) / k) : 0.0;
      const double pj = sj ? static_cast<double>(dj[q]) / (static_cast<double>(sj) / k) : 0.0;
      acc += (pi - pj) * (pi - pj);
    }
  }
  acc = wave_sum_d(acc);
  if (lane == 0) dred[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += dred[w];
    dist[static_cast<int64_t>(i) * F + j] = sqrt(s);
    dist[static_cast<int64_t>(j) * F + i] = sqrt(s);
  }
}

constexpr int kTopWaves = kTopThreads / 64;
constexpr int kRowPairs = TACG_MAX_EXPERTS / 2 / kTopWaves;  // row pairs per wave

// Inclusive prefix sum over the wave.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(v, o, 64);
    if ((threadIdx.x & 63) >= o) v += t;
  }
  return v;
}

__device__ __forceinline__ uint64_t low_lanes(int n) { return n >= 64 ? ~0ull : n <= 0 ? 0ull : (1ull << n) - 1ull; }

constexpr int kList = 2048;  // values searched by one wave
static_assert(kList >= kTopThreads, "the list also holds the threads' maxima");

// The largest t in [lo, hi] with at least n of the wave's values at or above it; lo if there is none.
template <int M>
__device__ __forceinline__ uint32_t largest_with(const uint32_t (&m)[M], uint32_t lo, uint32_t hi, uint32_t n) {
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo + 1u) / 2u;
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < M; ++i) c += __popcll(__ballot(m[i] >= mid));
    if (c >= n) lo = mid;
    else hi = mid - 1u;
  }
  return lo;
}

template <int NQ>  // dwords per lane and row pair: ceil((E - 1) / 64)
__global__ __launch_bounds__(kTopThreads) void top_pairs_kernel(const uint32_t* __restrict__ C, int F, int L, int E,
                                                                int top_n, int32_t* __restrict__ out) {
  __shared__ uint32_t red[2][kTopWaves];
  __shared__ uint32_t n_gt[TACG_MAX_EXPERTS], n_eq[TACG_MAX_EXPERTS];     // per row: counts above T, at T
  __shared__ uint32_t take[TACG_MAX_EXPERTS], base[TACG_MAX_EXPERTS];     // per row: ties to keep, first slot
  __shared__ uint32_t list[kList], n_list, range[2], n_chosen;
  const int f = blockIdx.x, l = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t n = static_cast<uint32_t>(top_n);
  const int n_pairs = (E + 1) / 2;  // row pairs (a, E - 1 - a); of an odd E's middle row only itself
  const uint32_t* seg = C + (static_cast<int64_t>(f) * L + l) * E * static_cast<int64_t>(E);
  // entry k of row pair a: column a + 1 + k of row a, then (k >= E - 1 - a) the columns of row E - 1 - a
  uint32_t v[kRowPairs][NQ];
  uint32_t mx = 0;
#pragma unroll
  for (int r = 0; r < kRowPairs; ++r) {
    const int a = wave + kTopWaves * r, la = E - 1 - a;
    const int total = a >= n_pairs ? 0 : 2 * a == E - 1 ? la : E - 1;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int k = lane + 64 * q;
      const int at = k < la ? a * E + a + 1 + k : la * E + (la + 1) + (k - la);
      const uint32_t x = __builtin_nontemporal_load(seg + (k < total ? at : 0));
      v[r][q] = k < total ? x : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < kRowPairs; ++r)
#pragma unroll
    for (int q = 0; q < NQ; ++q) mx = max(mx, v[r][q]);
  list[tid] = mx;
  if (tid == 0) n_list = 0;
  __syncthreads();
  // T = the largest threshold >= 1 with at least top_n pairs at or above it (1 if fewer exist).  A first bound comes from
  // the threads' maxima alone: top_n of them at or above it are top_n pairs.
  if (wave == 0) {
    uint32_t m[kTopWaves], top = 0;
#pragma unroll
    for (int i = 0; i < kTopWaves; ++i) {
      m[i] = list[lane + 64 * i];
      top = max(top, m[i]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
    const uint32_t t0 = largest_with(m, 1u, max(top, 1u), n);
    if (lane == 0) {
      range[0] = t0;
      range[1] = max(top, 1u);
    }
  }
  __syncthreads();
  // the pairs at or above it, usually a few more than top_n, go to a list that one wave searches
  uint32_t lo = range[0], hi = range[1];
  {
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < kRowPairs; ++r)
#pragma unroll
      for (int q = 0; q < NQ; ++q) c += __popcll(__ballot(v[r][q] >= lo));
    uint32_t at = 0;
    if (c != 0) {
      if (lane == 0) at = atomicAdd(&n_list, c);
      at = __shfl(at, 0, 64);
#pragma unroll
      for (int r = 0; r < kRowPairs; ++r)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const uint64_t on = __ballot(v[r][q] >= lo);
          if (on == 0) continue;
          const uint32_t slot = at + __popcll(on & low_lanes(lane));
          if (v[r][q] >= lo && slot < kList) list[slot] = v[r][q];
          at += __popcll(on);
        }
    }
  }
  barrier_after_lds_atomics();
  if (n_list <= kList) {
    if (wave == 0) {
      uint32_t m[kList / 64];
#pragma unroll
      for (int i = 0; i < kList / 64; ++i) m[i] = lane + 64 * i < n_list ? list[lane + 64 * i] : 0u;
      lo = largest_with(m, lo, hi, n);
      if (lane == 0) range[0] = lo;
    }
    __syncthreads();
    lo = range[0];
  } else {  // many ties: all waves search their registers
    for (int it = 0; lo < hi; it ^= 1) {  // the two buffers of the waves' counts alternate: one barrier a step
      const uint32_t mid = lo + (hi - lo + 1u) / 2u;
      uint32_t c = 0;
#pragma unroll
      for (int r = 0; r < kRowPairs; ++r)
#pragma unroll
        for (int q = 0; q < NQ; ++q) c += __popcll(__ballot(v[r][q] >= mid));
      if (lane == 0) red[it][wave] = c;
      __syncthreads();
      c = 0;
#pragma unroll
      for (int w = 0; w < kTopWaves; ++w) c += red[it][w];
      if (c >= n) lo = mid;
      else hi = mid - 1u;
    }
  }
  const uint32_t T = lo;
  // every row's pairs above T and at T (each row belongs to one row pair)
#pragma unroll
  for (int r = 0; r < kRowPairs; ++r) {
    const int a = wave + kTopWaves * r, la = E - 1 - a;
    if (a >= n_pairs) continue;
    uint32_t ga = 0, gb = 0, ea = 0, eb = 0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (__ballot(v[r][q] >= T) == 0) continue;  // nearly always, for a small top_n
      const uint64_t g = __ballot(v[r][q] > T), e = __ballot(v[r][q] == T), m = low_lanes(la - 64 * q);
      ga += __popcll(g & m);
      gb += __popcll(g & ~m);
      ea += __popcll(e & m);
      eb += __popcll(e & ~m);
    }
    if (lane == 0) {
      if (la != a) {
        n_gt[la] = gb;
        n_eq[la] = eb;
      }
      n_gt[a] = ga;
      n_eq[a] = ea;
    }
  }
  __syncthreads();
  if (wave == 0) {
    uint32_t g[4], e[4], sg = 0, se = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // rows 4 lane .. 4 lane + 3
      const int row = 4 * lane + i;
      g[i] = row < E ? n_gt[row] : 0u;
      e[i] = row < E ? n_eq[row] : 0u;
      sg += g[i];
      se += e[i];
    }
    const uint32_t above = __shfl(wave_scan(sg), 63, 64);  // below top_n
    const uint32_t upto = wave_scan(se);
    uint32_t ties = upto - se;  // at T in the rows before
    const uint32_t need = min(n, above + __shfl(upto, 63, 64)) - above;
    uint32_t chosen = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t t = ties < need ? min(e[i], need - ties) : 0u;
      ties += e[i];
      if (4 * lane + i < E) take[4 * lane + i] = t;
      g[i] += t;
      chosen += g[i];
    }
    const uint32_t end = wave_scan(chosen);
    uint32_t at = end - chosen;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (4 * lane + i < E) base[4 * lane + i] = at;
      at += g[i];
    }
    if (lane == 63) n_chosen = end;
  }
  __syncthreads();
  int32_t* dst = out + (static_cast<int64_t>(f) * L + l) * top_n;
  const uint64_t below = low_lanes(lane);
#pragma unroll
  for (int r = 0; r < kRowPairs; ++r) {
    const int a = wave + kTopWaves * r, la = E - 1 - a;
    if (a >= n_pairs) continue;
    uint32_t slot_a = base[a], slot_b = base[la], left_a = take[a], left_b = take[la];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (__ballot(v[r][q] >= T) == 0) continue;
      const uint64_t e = __ballot(v[r][q] == T), m = low_lanes(la - 64 * q);
      const bool in_a = (m >> lane) & 1ull;
      const uint64_t mine = in_a ? m : ~m;
      const uint32_t left = in_a ? left_a : left_b;
      const bool pick = v[r][q] > T || (v[r][q] == T && static_cast<uint32_t>(__popcll(e & mine & below)) < left);
      const uint64_t c = __ballot(pick);
      if (pick) {
        const int k = lane + 64 * q;
        const uint32_t slot = (in_a ? slot_a : slot_b) + __popcll(c & mine & below);
        dst[slot] = in_a ? a * E + a + 1 + k : la * E + la + 1 + (k - la);
      }
      slot_a += __popcll(c & m);
      slot_b += __popcll(c & ~m);
      left_a -= min(left_a, static_cast<uint32_t>(__popcll(e & m)));
      left_b -= min(left_b, static_cast<uint32_t>(__popcll(e & ~m)));
    }
  }
  for (uint32_t s = n_chosen + tid; s < n; s += kTopThreads) dst[s] = -1;
}

// number of entries >= 0 of a list padded with -1
__device__ __forceinline__ int list_len(const int32_t* v, int n) {
  int lo = 0, hi = n;  // first index holding -1 (the valid entries come first)
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (v[mid] >= 0) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(64) void jaccard_kernel(const int32_t* __restrict__ pairs, int F, int L, int top_n,
                                                     double* __restrict__ jac) {
  const int l = blockIdx.x, i = blockIdx.y, j = blockIdx.z;
  if (i > j) return;  // written with (j, i)
  const int32_t* a = pairs + (static_cast<int64_t>(i) * L + l) * top_n;
  const int32_t* b = pairs + (static_cast<int64_t>(j) * L + l) * top_n;
  const int na = list_len(a, top_n), nb = list_len(b, top_n);
  int inter = 0;
  for (int q = threadIdx.x; q < na; q += 64) {
    const int32_t x = a[q];
    int lo = 0, hi = nb;
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (b[mid] < x) lo = mid + 1;
      else hi = mid;
    }
    inter += (lo < nb && b[lo] == x) ? 1 : 0;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) inter += __shfl_xor(inter, o, 64);
  if (threadIdx.x == 0) {
    const int uni = na + nb - inter;
    const double x = uni ? static_cast<double>(inter) / uni : 1.0;
    jac[(static_cast<int64_t>(l) * F + i) * F + j] = x;
    jac[(static_cast<int64_t>(l) * F + j) * F + i] = x;
  }
}

}  // namespace

int launch_activation_distance(const uint32_t* D, int32_t F, int32_t L, int32_t E, int32_t k, double* dist,
                               hipStream_t stream) {
  // a wave per layer; more waves than layers only delay the launch (33 families, E = 33, one layer: 5.6 us with 16 waves, 4.1 with 4)
  const int waves = std::min(kDistThreads / 64, std::max(4, L));
  hipLaunchKernelGGL(dist_kernel, dim3(F, F), dim3(64 * waves), 0, stream, D, F, L, E, k, dist);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

int launch_pair_jaccard(const uint32_t* C, int32_t F, int32_t L, int32_t E, int32_t top_n, int32_t* top_pairs,
                        double* jaccard, hipStream_t stream) {
  const dim3 grid(F, L), block(kTopThreads);
  switch ((E + 62) / 64) {
    case 1: hipLaunchKernelGGL(top_pairs_kernel<1>, grid, block, 0, stream, C, F, L, E, top_n, top_pairs); break;
    case 2: hipLaunchKernelGGL(top_pairs_kernel<2>, grid, block, 0, stream, C, F, L, E, top_n, top_pairs); break;
    case 3: hipLaunchKernelGGL(top_pairs_kernel<3>, grid, block, 0, stream, C, F, L, E, top_n, top_pairs); break;
    default: hipLaunchKernelGGL(top_pairs_kernel<4>, grid, block, 0, stream, C, F, L, E, top_n, top_pairs); break;
  }
  hipLaunchKernelGGL(jaccard_kernel, dim3(L, F, F), dim3(64), 0, stream, top_pairs, F, L, top_n, jaccard);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

}  // namespace tacg
