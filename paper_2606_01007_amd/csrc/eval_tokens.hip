// Placement scoring for few placements (eval_uses_tokens): the trace pass of tacg_eval_placements and
// tacg_eval_trace_stats with lane = token.
//
// The lane = placement pass (eval.hip) scores 128 placements per wave whatever their number, and walks the
// tokens one by one.  Here a wave takes 64 tokens at once, one per lane, and up to four placements together: LDS
// row tbl[e] holds the four placements' one-hot GPU masks of expert e (zero where it has several candidates), so a slot
// costs a lane one 16-byte read.  The replicated slots of a token are resolved in slot order from the rows
// rinfo[r] = (feasible candidates, least-loaded) of the four placements, all lanes stepping to their i-th such slot
// together, and their choices are LDS counters.  A workgroup takes a chunk of one family's tokens of one layer
// and four placements.
//
// What bounds it, from its instructions (no counters): the LDS, whose reads go to random rows (one expert per lane).  Measured on MI355X: two
// placements of E = 256, top-8, 32 GPUs, 16 x 3 replicas, 2^19 tokens x 58 layers with the per-token statistics:
// 4.59 -> 0.43 ms for the whole call.
#include "eval_internal.h"

namespace tacg {
namespace {

constexpr int kThreads = 512;
constexpr int kPB = 4;                   // placements per workgroup
constexpr int64_t kMinChunk = 4096, kMaxChunk = int64_t(1) << 20;  // tokens per workgroup

struct TkFam {  // 16-byte records (runtime-indexed kernel arguments)
  uint32_t off, end, first_piece, band;  // band: home_start | home_size << 8
};

struct TkArgs {
  const int16_t* trace;
  const uint8_t* primary;
  EvWs ws;
  int64_t N;
  int32_t L, E, F, G, P;
  int32_t n_pieces, n_pblocks, stats;
  uint32_t chunk, band_starts;
  TkFam fam[TACG_MAX_FAMILIES + 1];
};
static_assert(sizeof(TkArgs) <= 4096, "kernel arguments must stay within 4 KB");

// grid (layers x pieces x placement blocks, placement block fastest)
template <int K>
__global__ __launch_bounds__(kThreads) void ev_tokens(TkArgs a) {
  __shared__ uint4 tbl[TACG_MAX_EXPERTS + 1];                        // one-hot masks of the four placements; row E is zero
  __shared__ uint4 rinfo[TACG_MAX_REPLICATED][kPB / 2];              // (FC, least-loaded) of placements 0, 1 and 2, 3
  __shared__ uint32_t rcnt[kPB][TACG_MAX_GPUS];                      // choices of replicated slots
  __shared__ uint32_t red[3][kPB], n_ok;                             // |cards|, cards but the anchor, tokens over several bands
  __shared__ uint8_t rep_of[TACG_MAX_EXPERTS + 1];
  const int E = a.E, L = a.L, P = a.P;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kWaves = kThreads / 64;
  const uint32_t total = gridDim.x, b = blockIdx.x;  // XCD-aware order, as in ev_main
  const uint32_t xcd = b % kXcds, per = total / kXcds, rem = total % kXcds;
  const uint32_t vid = xcd * per + min(xcd, rem) + b / kXcds;
  const int pb = static_cast<int>(vid % a.n_pblocks);
  const uint32_t lp = vid / a.n_pblocks;
  const uint32_t piece = lp % a.n_pieces;
  const int l = lp / a.n_pieces;
  const int p0 = pb * kPB, npl = min(kPB, P - p0);
  int f = 0;
  while (a.fam[f + 1].first_piece <= piece) ++f;
  const TkFam fr = a.fam[f];
  const uint32_t hs = fr.band & 0xffu, hz = fr.band >> 8;
  const uint32_t t0 = fr.off + (piece - fr.first_piece) * a.chunk;
  const uint32_t n = min(fr.end - t0, a.chunk);  // tokens are counted from t0: t0 + chunk may pass 2^32

  // ---- tables ----
  const int nrep = a.ws.n_rep[l];
  if (tid <= E) {
    uint32_t m[kPB] = {};
    uint8_t r = kNone;
    if (tid < E) {
      r = a.ws.rep_of[static_cast<int64_t>(l) * E + tid];
#pragma unroll
      for (int q = 0; q < kPB; ++q) {
        const int p = p0 + min(q, npl - 1);
        const uint32_t g = a.primary[(static_cast<int64_t>(p) * L + l) * E + tid];
        bool single = q < npl && g < static_cast<uint32_t>(a.G);
        if (r != kNone)
          single = single && (a.ws.rep_info[(static_cast<int64_t>(l) * TACG_MAX_REPLICATED + r) * P + p].y >> 31);
        m[q] = single ? 1u << g : 0u;
      }
    }
    tbl[tid] = make_uint4(m[0], m[1], m[2], m[3]);
    rep_of[tid] = r;
  }
  for (int i = tid; i < nrep * kPB; i += kThreads) {
    const int r = i / kPB, q = i % kPB;
    const uint2 v = a.ws.rep_info[(static_cast<int64_t>(l) * TACG_MAX_REPLICATED + r) * P + p0 + min(q, npl - 1)];
    reinterpret_cast<uint2*>(rinfo[r])[q] = make_uint2(v.x, v.y & 31u);
  }
  if (tid < kPB * TACG_MAX_GPUS) rcnt[tid / TACG_MAX_GPUS][tid % TACG_MAX_GPUS] = 0;
  if (tid < 3 * kPB) red[tid / kPB][tid % kPB] = 0;
  if (tid == 0) n_ok = 0;
  __syncthreads();

  const bool any_bad = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(*a.ws.n_bad != 0u)) != 0u;
  const int16_t* trace_c = a.trace + (static_cast<int64_t>(l) * a.N + t0) * K;
  const uint32_t pos0 = t0 - fr.off;
  uint32_t span[kPB] = {}, away[kPB] = {}, cross[kPB] = {}, scored = 0;
  TraceIds<K> next;  // the next tile's ids are in flight while one is scored
  next.fetch(trace_c + static_cast<int64_t>(min(static_cast<uint32_t>(tid), n - 1)) * K);
  for (uint32_t tile = wave * 64; tile < n; tile += kThreads) {
    const uint32_t t = tile + lane;
    uint32_t id[K];
    next.unpack(id);
    next.fetch(trace_c + static_cast<int64_t>(min(t + kThreads, n - 1)) * K);
    bool ok = t < n;
    if (any_bad) {  // some token-layer of the trace is invalid: leave those out
      bool dup = false;
#pragma unroll
      for (int s = 0; s < K; ++s) {
        ok &= id[s] < static_cast<uint32_t>(E);
#pragma unroll
        for (int q = 0; q < s; ++q) dup |= id[s] == id[q];
      }
      ok &= !dup;
    }
    scored += ok ? 1u : 0u;
    const uint32_t h = hs + (pos0 + t) % hz;
    uint32_t m[kPB] = {};
    uint64_t reps = 0;  // the replicated slots' indices in slot order, four bits each
    uint32_t cnt = 0;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const uint32_t e = ok ? id[s] : static_cast<uint32_t>(E);
      const uint4 v = tbl[e];
      m[0] |= v.x;
      m[1] |= v.y;
      m[2] |= v.z;
      m[3] |= v.w;
      if (nrep > 0) {
        const uint32_t r = rep_of[e];
        const bool is = r != kNone;
        reps |= static_cast<uint64_t>(is ? r : 0u) << (4 * cnt);
        cnt += is ? 1u : 0u;
      }
    }
    for (uint32_t i = 0; __any(i < cnt); ++i) {  // at most K steps
      const uint32_t r = static_cast<uint32_t>(reps) & 15u;
      reps >>= 4;
      if (i < cnt) {
        uint2 v[kPB];
#pragma unroll
        for (int q = 0; q < kPB; q += 2) {
          const uint4 x = rinfo[r][q / 2];
          v[q] = make_uint2(x.x, x.y);
          v[q + 1] = make_uint2(x.z, x.w);
        }
#pragma unroll
        for (int q = 0; q < kPB; ++q) {
          if (q >= npl) break;
          // the lowest feasible candidate the token reaches, else the anchor if feasible, else the least-loaded
          const uint32_t x = v[q].x & m[q];
          const uint32_t alt = ((v[q].x >> h) & 1u) ? h : v[q].y;
          const uint32_t pick = x != 0u ? static_cast<uint32_t>(__builtin_ctz(x)) : alt;
          m[q] |= 1u << pick;
          __hip_atomic_fetch_add(&rcnt[q][pick], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < kPB; ++q) {
      span[q] += __popc(m[q]);
      away[q] += __popc(m[q] & ~(1u << h));
      if (a.stats) {
        // the cards lie in more than one band exactly when a band starts in (lowest card, highest card] (see ev_main)
        const uint32_t lo = static_cast<uint32_t>(__builtin_ctz(m[q] | 0x80000000u));
        const uint32_t top = 0x80000000u >> (__builtin_clz(m[q] | 1u) & 31);
        const uint32_t range = (top << 1) + (0xfffffffeu << lo);
        cross[q] += (m[q] != 0u && (a.band_starts & range) != 0u) ? 1u : 0u;
      }
    }
  }

  // ---- flush ----
#pragma unroll
  for (int q = 0; q < kPB; ++q) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      span[q] += __shfl_xor(span[q], o, 64);
      away[q] += __shfl_xor(away[q], o, 64);
      cross[q] += __shfl_xor(cross[q], o, 64);
    }
    if (lane == 0) {
      atomicAdd(&red[0][q], span[q]);
      atomicAdd(&red[1][q], away[q]);
      atomicAdd(&red[2][q], cross[q]);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) scored += __shfl_xor(scored, o, 64);
  if (lane == 0) atomicAdd(&n_ok, scored);
  barrier_after_lds_atomics();
  if (tid < npl) {
    const int p = p0 + tid;
    const int64_t fp = static_cast<int64_t>(f) * P + p;
    atomicAdd(&a.ws.acc_span[p], static_cast<unsigned long long>(red[0][tid]));
    atomicAdd(&a.ws.acc_home[p], static_cast<unsigned long long>(red[1][tid]));
    atomicAdd(&a.ws.acc_fam[fp], static_cast<unsigned long long>(red[1][tid]));
    if (a.stats) {  // |cards| - 1 summed over the tokens (each scored one has at least one card)
      atomicAdd(&a.ws.acc_span_fam[fp], static_cast<unsigned long long>(red[0][tid] - n_ok));
      atomicAdd(&a.ws.acc_cross_fam[fp], static_cast<unsigned long long>(red[2][tid]));
    }
  }
  if (tid < npl * a.G) {
    const int q = tid / a.G, g = tid % a.G;
    const uint32_t c = rcnt[q][g];
    if (c) {
      atomicAdd(a.ws.rep_load + (static_cast<int64_t>(l) * a.G + g) * even_up(P) + p0 + q, c);
      if (a.stats && static_cast<uint32_t>(g) - hs < hz)  // served inside the family's own band
        atomicAdd(a.ws.acc_hmass_fam + static_cast<int64_t>(f) * P + p0 + q, static_cast<unsigned long long>(c));
    }
  }
}

template <int K>
int launch_t(const TkArgs& a, hipStream_t stream) {
  const int64_t grid = static_cast<int64_t>(a.n_pblocks) * a.n_pieces * a.L;
  if (grid > 0x7fffffff) return TACG_E_UNSUPPORTED;
  hipLaunchKernelGGL(ev_tokens<K>, dim3(static_cast<uint32_t>(grid)), dim3(kThreads), 0, stream, a);
  return TACG_OK;
}

}  // namespace

int launch_eval_tokens(const EvBase& e, const int64_t* fam_off_host, const int32_t* home_start_host,
                       const int32_t* home_size_host, hipStream_t stream) {
  TkArgs a{};
  a.trace = e.trace;
  a.primary = e.primary;
  a.ws = e.ws;
  a.N = e.N;
  a.L = e.L;
  a.E = e.E;
  a.F = e.F;
  a.G = e.G;
  a.P = e.P;
  a.stats = e.stats;
  a.band_starts = e.band_starts;
  a.n_pblocks = (e.P + kPB - 1) / kPB;
  // about eight workgroups per CU
  int64_t chunk = (e.N * e.L * a.n_pblocks + 2047) / 2048;
  chunk = std::min(kMaxChunk, std::max(kMinChunk, (chunk + kThreads - 1) / kThreads * kThreads));
  a.chunk = static_cast<uint32_t>(chunk);
  int64_t np = 0;
  for (int f = 0; f < e.F; ++f) {
    a.fam[f] = TkFam{static_cast<uint32_t>(fam_off_host[f]), static_cast<uint32_t>(fam_off_host[f + 1]),
                     static_cast<uint32_t>(np),
                     static_cast<uint32_t>(home_start_host[f]) | (static_cast<uint32_t>(home_size_host[f]) << 8)};
    np += (fam_off_host[f + 1] - fam_off_host[f] + chunk - 1) / chunk;
  }
  for (int f = e.F; f <= TACG_MAX_FAMILIES; ++f) a.fam[f] = TkFam{0u, 0u, 0xffffffffu, 1u << 8};
  if (np > 0x7fffffff) return TACG_E_UNSUPPORTED;
  a.n_pieces = static_cast<int32_t>(np);
  if (np == 0) return TACG_OK;
  switch (e.K) {
#define TACG_K(k) \
  case k:         \
    return launch_t<k>(a, stream);
    TACG_K(1) TACG_K(2) TACG_K(3) TACG_K(4) TACG_K(5) TACG_K(6) TACG_K(7) TACG_K(8)
    TACG_K(9) TACG_K(10) TACG_K(11) TACG_K(12) TACG_K(13) TACG_K(14) TACG_K(15) TACG_K(16)
#undef TACG_K
    default:
      return TACG_E_UNSUPPORTED;
  }
}

}  // namespace tacg
