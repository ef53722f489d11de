// Family preferences and the task-modulated co-activation graph (Sec. 3.3, eqs.
// usage-coact-advantage, coact-advantage, zscore, soft-score, family-pref, same-family-kernel,
// task-modulated-graph).  Internal arithmetic is float64; outputs are float32.
//
// Three passes per call (all small next to the trace passes; C is read once):
//   rw_rows   grid (L, row blocks): per row i and family f the co-activation strength
//             c_f(i) = sum_{j != i} C_f[i][j] / N_f, the pooled A-bar[i][j] = mean_f C_f[i][j] / N_f
//             (zero diagonal) and the row block's maximum of A-bar.  A wave per eight families, summed by halving
//             exchanges; the next row's loads are in flight.
//   rw_pref   grid (L): usage u_f = D_f / (N_f k), advantages against the mean of the other families, z-scores over
//             experts (population std; a wave per family), s = z(du) + z(dc), the softmax over f of the
//             layer's scores and the layer maximum of A-bar.
//   rw_graph  grid (L, row blocks): A-hat = A-bar / max, A_task = P P^T, A-tilde; a wave holds four rows x four
//             columns per lane, so each preference read from LDS serves four products.
// Bound by the read of C (rw_rows: 243 MB at E = 256, 16 families, 58 layers).  Measured on MI355X at that size, whole
// call: 119 -> 102 us (a pass of its own for N_f, the softmax repeated in every row block of the graph
// pass, a preference read per product).
#include "tacg_internal.h"

namespace tacg {
namespace {

constexpr int kRows = 16;  // most rows of a layer per workgroup (rw_graph: always)

struct RwWs {
  double* c;          // [L][F][E]
  double* abar;       // [L][E][E]
  double* max;        // [L]        maximum of A-bar
  double* s;          // [L][F][E]  maxima of the row blocks (from the layer's first entry on), then preferences
};

RwWs carve_rw(void* ws, int32_t F, int32_t L, int32_t E, size_t* used = nullptr) {
  Carver c{static_cast<char*>(ws), 0};
  RwWs r;
  r.c = c.take<double>(static_cast<size_t>(L) * F * E);
  r.abar = c.take<double>(static_cast<size_t>(L) * E * E);
  r.max = c.take<double>(static_cast<size_t>(L));
  r.s = c.take<double>(static_cast<size_t>(L) * F * E);
  if (used) *used = c.used;
  return r;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

constexpr int kSums = 8;  // values summed over the wave together, and most family rows of C held by a wave

// One halving exchange between lanes 8 M apart: the lower lane keeps values 0 .. M - 1 of both, the upper one M .. 2 M - 1.
template <int M>
__device__ __forceinline__ void halve(double* x) {
  const bool up = (threadIdx.x & (8 * M)) != 0;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const double keep = up ? x[i + M] : x[i], send = up ? x[i] : x[i + M];
    x[i] = keep + __shfl_xor(send, 8 * M, 64);
  }
}

// Sums x[0..7] over the wave: every lane gets the sum of value (lane >> 3) & 7.  Ten exchanges against 48 for
// eight separate sums.
__device__ __forceinline__ double wave_sum8(double (&x)[kSums]) {
  halve<4>(x);
  halve<2>(x);
  halve<1>(x);
  double s = x[0];
  s += __shfl_xor(s, 4, 64);
  s += __shfl_xor(s, 2, 64);
  s += __shfl_xor(s, 1, 64);
  return s;
}

// N_f of the layer's families into nf: one wave per family, an exact integer sum over the experts.  The caller
// synchronises.
__device__ __forceinline__ void family_tokens(const uint32_t* __restrict__ D, int F, int L, int E, int k, int l,
                                              double* nf) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int f = wave; f < F; f += nw) {
    const uint32_t* d = D + (static_cast<int64_t>(f) * L + l) * E;
    unsigned long long t = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = lane + 64 * q;
      if (e < E) t += d[e];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o, 64);
    if (lane == 0) nf[f] = static_cast<double>(t) / k;
  }
}

// One wave's share of the family rows of C: families f0 .. f0 + U - 1 (f0 = 8 wave) of a row, four columns per lane.  U = 2 or
// 4 for at most so many families in all (E = 256, 2 families, 58 layers, GESR scores: 35.6 us with the arithmetic of eight).
template <int U>
struct FamRows {
  double inv[U];           // 1 / N_f (0 for an empty family or past F)
  const uint32_t* base;    // row 0 of family f0
  int64_t stride;          // between families
  int E, n;                // n: families of this wave
  uint32_t next[U][4];

  __device__ __forceinline__ void init(const uint32_t* D, const uint32_t* C, int F, int L, int E_, int k, int l, int f0) {
    const int lane = threadIdx.x & 63;
    E = E_;
    n = min(U, F - f0);
    stride = static_cast<int64_t>(L) * E * E;
    base = C + (static_cast<int64_t>(f0) * L + l) * E * E;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t* d = D + (static_cast<int64_t>(f0 + min(u, n - 1)) * L + l) * E;
      unsigned long long t = 0;  // an exact integer sum over the experts
#pragma unroll
      for (int q = 0; q < 4; ++q) t += lane + 64 * q < E ? d[min(lane + 64 * q, E - 1)] : 0u;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o, 64);
      const double nf = static_cast<double>(t) / k;
      inv[u] = u < n && nf > 0 ? 1.0 / nf : 0.0;
    }
  }
  __device__ __forceinline__ void fetch(int i) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t* row = base + min(u, n - 1) * stride + static_cast<int64_t>(i) * E;
#pragma unroll
      for (int q = 0; q < 4; ++q) next[u][q] = row[min(lane + 64 * q, E - 1)];
    }
  }
  // the fetched rows, the diagonal and columns past E as zero
  __device__ __forceinline__ void take(int i, uint32_t (&v)[U][4]) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool on = lane + 64 * q < E && lane + 64 * q != i;
#pragma unroll
      for (int u = 0; u < U; ++u) v[u][q] = on ? next[u][q] : 0u;
    }
  }
};

// Workgroups of ceil(F / 8) waves, one row of A-bar at a time: every wave scales its families' rows, the waves' parts of
// the row meet in LDS (two buffers in turn, one barrier a row), and the next row's loads are in flight meanwhile.
// grid (L, row blocks); dynamic LDS: 2 x waves x E doubles.
template <int U>
__global__ __launch_bounds__(512) void rw_rows(const uint32_t* __restrict__ D, const uint32_t* __restrict__ C, int F,
                                               int L, int E, int k, int rows, RwWs ws) {
  extern __shared__ double part[];  // [2][nw][E]
  __shared__ double wmax[TACG_MAX_FAMILIES / kSums];
  const int l = blockIdx.x, nw = blockDim.x >> 6;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = blockIdx.y * rows, r1 = min(E, r0 + rows);
  FamRows<U> fr;
  fr.init(D, C, F, L, E, k, l, kSums * wave);
  fr.fetch(r0);
  double mx = 0.0;
  for (int i = r0; i < r1; ++i) {
    uint32_t v[U][4];
    fr.take(i, v);
    fr.fetch(min(i + 1, E - 1));
    double* const mine = part + static_cast<size_t>(((i & 1) * nw + wave)) * E;
    double x[kSums] = {}, ab[4] = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      x[u] = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double a = v[u][q] * fr.inv[u];
        x[u] += a;
        ab[q] += a;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (lane + 64 * q < E) mine[lane + 64 * q] = ab[q];
    const double c = wave_sum8(x);
    if ((lane & 7) == 0 && (lane >> 3) < fr.n)
      ws.c[(static_cast<int64_t>(l) * F + kSums * wave + (lane >> 3)) * E + i] = c;
    __syncthreads();
    const double* const all = part + static_cast<size_t>((i & 1) * nw) * E;
    for (int j = threadIdx.x; j < E; j += blockDim.x) {
      double t = 0.0;
      for (int w = 0; w < nw; ++w) t += all[w * E + j];
      t /= F;
      ws.abar[(static_cast<int64_t>(l) * E + i) * E + j] = t;
      mx = fmax(mx, t);
    }
  }
  mx = wave_max(mx);
  if (lane == 0) wmax[wave] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < nw; ++w) mx = fmax(mx, wmax[w]);
    // a layer of s has F E >= 2 E entries, more than its row blocks
    ws.s[static_cast<int64_t>(l) * F * E + blockIdx.y] = mx;
  }
}

constexpr int kPrefThreads = 1024;

// One workgroup per layer.  LDS: scores [F][E], then per expert the sums over families [4][E] of u and of c.
__global__ __launch_bounds__(kPrefThreads) void rw_pref(const uint32_t* __restrict__ D, int F, int L, int E, int k,
                                                        double tau, double eps, int row_blocks, float* __restrict__ pref,
                                                        RwWs ws) {
  extern __shared__ double sc[];
  __shared__ double nf[TACG_MAX_FAMILIES];
  double* const sum_u = sc + static_cast<size_t>(F) * E;  // [4][E], then in [0][E] the maximum over f
  double* const sum_c = sum_u + 4 * static_cast<size_t>(E);  // [4][E], then in [0][E] the softmax denominator
  const int l = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  constexpr int kWaves = kPrefThreads / 64;
  double* const sl = ws.s + static_cast<int64_t>(l) * F * E;
  const double* const cl = ws.c + static_cast<int64_t>(l) * F * E;
  family_tokens(D, F, L, E, k, l, nf);
  if (wave == 0) {
    const double m = wave_max(lane < row_blocks ? sl[lane] : 0.0);  // at most 64 row blocks
    if (lane == 0) ws.max[l] = m;
  }
  __syncthreads();
  // sums over the families of every expert, a quarter of the families per thread
  const int e4 = tid & 255, part = tid >> 8;
  if (e4 < E) {
    double su = 0.0, scv = 0.0;
#pragma unroll 4
    for (int g = part; g < F; g += 4) {
      const double n = nf[g];
      su += n > 0 ? D[(static_cast<int64_t>(g) * L + l) * E + e4] / (n * k) : 0.0;
      scv += cl[g * E + e4];
    }
    sum_u[part * E + e4] = su;
    sum_c[part * E + e4] = scv;
  }
  __syncthreads();
  // soft scores, a wave per family
  for (int f = wave; f < F; f += kWaves) {
    const double n = nf[f];
    double du[4], dc[4], mu_u = 0.0, mu_c = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = lane + 64 * q;
      du[q] = dc[q] = 0.0;
      if (e < E) {
        const double uf = n > 0 ? D[(static_cast<int64_t>(f) * L + l) * E + e] / (n * k) : 0.0;
        const double cf = cl[f * E + e];
        const double su = (sum_u[e] + sum_u[E + e]) + (sum_u[2 * E + e] + sum_u[3 * E + e]);
        const double scv = (sum_c[e] + sum_c[E + e]) + (sum_c[2 * E + e] + sum_c[3 * E + e]);
        du[q] = uf - (su - uf) / (F - 1);
        dc[q] = cf - (scv - cf) / (F - 1);
      }
      mu_u += du[q];
      mu_c += dc[q];
    }
    mu_u = wave_sum(mu_u) / E;
    mu_c = wave_sum(mu_c) / E;
    double vu = 0.0, vc = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (lane + 64 * q < E) {
        vu += (du[q] - mu_u) * (du[q] - mu_u);
        vc += (dc[q] - mu_c) * (dc[q] - mu_c);
      }
    }
    const double su = sqrt(wave_sum(vu) / E) + eps, sv = sqrt(wave_sum(vc) / E) + eps;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = lane + 64 * q;
      if (e < E) sc[f * E + e] = ((du[q] - mu_u) / su + (dc[q] - mu_c) / sv) / tau;
    }
  }
  __syncthreads();
  // softmax over the families: maximum, exponentials, denominator
  if (tid < E) {
    double m = -INFINITY;
    for (int f = 0; f < F; ++f) m = fmax(m, sc[f * E + tid]);
    sum_u[tid] = m;
  }
  __syncthreads();
  for (int i = tid; i < F * E; i += kPrefThreads) sc[i] = exp(sc[i] - sum_u[i % E]);
  __syncthreads();
  if (tid < E) {
    double d = 0.0;
    for (int f = 0; f < F; ++f) d += sc[f * E + tid];
    sum_c[tid] = d;
  }
  __syncthreads();
  for (int i = tid; i < F * E; i += kPrefThreads) {
    const int f = i / E, e = i - f * E;
    const double p = sc[i] / sum_c[e];
    sl[i] = p;
    pref[(static_cast<int64_t>(l) * E + e) * F + f] = static_cast<float>(p);
  }
}

__global__ __launch_bounds__(256, 4) void rw_graph(int F, int L, int E, double alpha, float* __restrict__ a_tilde,
                                                   float* __restrict__ a_hat, RwWs ws) {
  extern __shared__ __align__(16) double P[];  // [F][E] preferences of the layer
  const int l = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  static_assert(kRows == 16, "four rows per wave");
  const int r0 = blockIdx.y * kRows + 4 * wave;
  const double* sl = ws.s + static_cast<int64_t>(l) * F * E;
  double ah[4][4];  // A-bar of this wave's rows, in flight while the preferences are staged
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      ah[r][q] = ws.abar[(static_cast<int64_t>(l) * E + min(r0 + r, E - 1)) * E + min(lane + 64 * q, E - 1)];
  for (int i = threadIdx.x; i < F * E; i += blockDim.x) P[i] = sl[i];
  __syncthreads();
  const double mx = ws.max[l];
  const double inv = mx > 0.0 ? 1.0 / mx : 0.0;
  double task[4][4] = {};
  for (int f = 0; f < F; ++f) {
    double pi[4], pj[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) pi[r] = P[f * E + min(r0 + r, E - 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) pj[q] = P[f * E + min(lane + 64 * q, E - 1)];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) task[r][q] += pi[r] * pj[q];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (r0 + r >= E) break;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = lane + 64 * q;
      if (j >= E) continue;
      const double h = mx > 0.0 ? ah[r][q] * inv : 0.0;
      const int64_t o = (static_cast<int64_t>(l) * E + r0 + r) * E + j;
      a_tilde[o] = static_cast<float>((1.0 - alpha) * h + alpha * (task[r][q] * h));
      if (a_hat) a_hat[o] = static_cast<float>(h);
    }
  }
}

// GESR identification scores (Sec. 3.4, eq. generic-score) per row i of layer l, float64:
// Cent = sum_j A-bar(i, j); Cons = mean_f cos(A_f(i, :), A-bar(i, :)) (0 for a zero row);
// Spec = max_f ||A_f(i, :) - A-bar(i, :)||_2.  The waves share a row as in rw_rows: a wave keeps its eight families'
// rows in registers between A-bar and the per-family terms, so C is read once.  Bound by the read of C (243 MB
// take 57 us here; by counters the waves wait 34 % of their time and the VALU is 51 % busy); measured on MI355X at E = 256, 16 families, 58 layers: 152 -> 70 us (C read twice, a wave sum per
// family and term).  grid (L, row blocks); dynamic LDS: 2 x waves x E doubles.
template <int U>
__global__ __launch_bounds__(512) void gesr_scores_kernel(const uint32_t* __restrict__ D, const uint32_t* __restrict__ C,
                                                          int F, int L, int E, int k, int rows,
                                                          double* __restrict__ cent, double* __restrict__ cons,
                                                          double* __restrict__ spec) {
  extern __shared__ double part[];  // [2][nw][E]
  constexpr int kMaxWaves = TACG_MAX_FAMILIES / kSums;
  __shared__ double row_cos[kRows][kMaxWaves], row_dev[kRows][kMaxWaves], row_sum[kRows];
  const int l = blockIdx.x, nw = blockDim.x >> 6;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = blockIdx.y * rows, r1 = min(E, r0 + rows);
  FamRows<U> fr;
  fr.init(D, C, F, L, E, k, l, kSums * wave);
  fr.fetch(r0);
  for (int i = r0; i < r1; ++i) {
    uint32_t v[U][4];
    fr.take(i, v);
    fr.fetch(min(i + 1, E - 1));
    double* const mine = part + static_cast<size_t>(((i & 1) * nw + wave)) * E;
    double ab[4] = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) ab[q] += v[u][q] * fr.inv[u];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (lane + 64 * q < E) mine[lane + 64 * q] = ab[q];
    __syncthreads();
    const double* const all = part + static_cast<size_t>((i & 1) * nw) * E;
    double cs = 0.0, nb2 = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ab[q] = 0.0;
      if (lane + 64 * q < E) {
        for (int w = 0; w < nw; ++w) ab[q] += all[w * E + lane + 64 * q];
        ab[q] /= F;
      }
      cs += ab[q];
      nb2 += ab[q] * ab[q];
    }
    const double nb = sqrt(wave_sum(nb2));
    double dot[kSums] = {}, na2[kSums] = {}, dev2[kSums] = {};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      dot[u] = na2[u] = dev2[u] = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        __asm__ __volatile__("" : "+v"(v[u][q]));  // scaled again, not kept in 64-bit registers since A-bar
        const double a = v[u][q] * fr.inv[u];
        dot[u] += a * ab[q];
        na2[u] += a * a;
        dev2[u] += (a - ab[q]) * (a - ab[q]);
      }
    }
    // lane 8 u holds the sums of family u
    const double d = wave_sum8(dot), n2 = wave_sum8(na2), e2 = wave_sum8(dev2);
    const bool on = (lane >> 3) < fr.n;
    const double na = sqrt(n2);
    double cos_sum = (on && na > 0.0 && nb > 0.0) ? d / (na * nb) : 0.0;
    double worst = on ? sqrt(e2) : 0.0;
#pragma unroll
    for (int o = 32; o >= 8; o >>= 1) {
      cos_sum += __shfl_xor(cos_sum, o, 64);
      worst = fmax(worst, __shfl_xor(worst, o, 64));
    }
    if (wave == 0) cs = wave_sum(cs);
    if (lane == 0) {
      row_cos[i - r0][wave] = cos_sum;
      row_dev[i - r0][wave] = worst;
      if (wave == 0) row_sum[i - r0] = cs;
    }
  }
  __syncthreads();
  const int r = threadIdx.x;
  if (r < r1 - r0) {
    double c = 0.0, w = 0.0;
    for (int u = 0; u < nw; ++u) {
      c += row_cos[r][u];
      w = fmax(w, row_dev[r][u]);
    }
    const int64_t o = static_cast<int64_t>(l) * E + r0 + r;
    cent[o] = row_sum[r];
    cons[o] = c / F;
    spec[o] = w;
  }
}

}  // namespace

size_t reweight_workspace(int32_t F, int32_t L, int32_t E) {
  size_t used = 0;
  carve_rw(nullptr, F, L, E, &used);
  return used;
}

// Rows per workgroup of the row passes: as few as leave no more workgroups than the chip holds at once at three waves per SIMD
// (a workgroup's rows are a chain; at 256 experts, 16 families, 58 layers 16 rows left the chip at 1.8 waves per SIMD and 8 made
// a round and a quarter), 16 at most.  GESR scores at 1, 2 and 4 rows: E = 8, 2 families, 24 layers 7.8, 9.9 and 15.0 us; E =
// 128, 16 families, 12 layers 12.7, 13.8 and 21.0; E = 256, 64 families, 4 layers (the chip full at 4) 43.6, 43.6 and 30.9.
static int rows_per_block(int L, int E, int nw) {
  const int64_t held = 256 * std::max(1, 12 / nw);
  int rows = 1;
  while (rows < kRows && static_cast<int64_t>(L) * ((E + rows - 1) / rows) > held) ++rows;
  return rows;
}

int launch_reweight(const uint32_t* D, const uint32_t* C, int32_t F, int32_t L, int32_t E, int32_t k,
                    double alpha, double tau, double eps, float* pref, float* a_tilde, float* a_hat,
                    void* workspace, hipStream_t stream) {
  RwWs ws = carve_rw(workspace, F, L, E);
  const int rb = (E + kRows - 1) / kRows;
  const size_t plds = static_cast<size_t>(F) * E * sizeof(double);  // <= 64 x 256 x 8 = 128 KB
  const size_t slds = plds + 8 * static_cast<size_t>(E) * sizeof(double);
  allow_lds(&rw_pref, slds, TACG_MAX_FAMILIES * sizeof(double));
  allow_lds(&rw_graph, plds);
  const int nw = (F + kSums - 1) / kSums;
  const int rows = std::max(rows_per_block(L, E, nw), (E + 63) / 64);  // rw_pref reads the blocks' maxima with one wave
  const int blocks = (E + rows - 1) / rows;
  auto* rows_kernel = F <= 2 ? &rw_rows<2> : F <= 4 ? &rw_rows<4> : &rw_rows<kSums>;
  hipLaunchKernelGGL(rows_kernel, dim3(L, blocks), dim3(64 * nw), 2 * static_cast<size_t>(nw) * E * sizeof(double), stream, D,
                     C, F, L, E, k, rows, ws);
  hipLaunchKernelGGL(rw_pref, dim3(L), dim3(kPrefThreads), slds, stream, D, F, L, E, k, tau, eps, blocks, pref, ws);
  hipLaunchKernelGGL(rw_graph, dim3(L, rb), dim3(256), plds, stream, F, L, E, alpha, a_tilde, a_hat, ws);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

int launch_gesr_scores(const uint32_t* D, const uint32_t* C, int32_t F, int32_t L, int32_t E, int32_t k, double* cent,
                       double* cons, double* spec, hipStream_t stream) {
  const int nw = (F + kSums - 1) / kSums, rows = rows_per_block(L, E, nw);
  auto* kernel = F <= 2 ? &gesr_scores_kernel<2> : F <= 4 ? &gesr_scores_kernel<4> : &gesr_scores_kernel<kSums>;
  hipLaunchKernelGGL(kernel, dim3(L, (E + rows - 1) / rows), dim3(64 * nw),
                     2 * static_cast<size_t>(nw) * E * sizeof(double), stream, D, C, F, L, E, k, rows, cent, cons, spec);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

}  // namespace tacg
