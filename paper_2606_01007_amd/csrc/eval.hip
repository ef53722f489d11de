// Placement scoring: per-token cross-GPU cost, GESR candidate choice and per-GPU loads
// (Sec. 3.4 serving rule with eqs. mean-load and feasible-set; App. C per-token dispatch sets;
// App. H "Comm"), plus the snapshot loads that feed the guard and Jain / MaxVio (App. H).
//
// Launch sequence of tacg_eval_placements:
//   ev_zero      clear the workspace accumulators
//   ev_flags     validate the placement tables; mark experts that have a secondary in any placement
//   ev_replist   per layer: compact index of the marked ("replicated") experts
//   ev_repinfo   per (placement, layer, replicated expert): feasible candidate mask FC, the
//                fallback GPU argmin_{m in FC} load_ref (ties: lowest number) and whether the expert
//                has a single candidate in that placement
//   ev_valid     validate the trace's ids: flag and count the token-layers with an id out of range
//                or a repeated id, and mark their groups of 64 token-layers; count every expert's dispatches
//   ev_main      the trace pass (below); an invalid token-layer (checked again only in marked groups) is not scored.  At
//                most 8 GPUs run on bit planes instead (eval_planes.hip), few placements with lane = token (eval_tokens.hip)
//   ev_finalize  loads = counts of single-candidate experts on their primary + replicated choices;
//                costs from the accumulators
//
// ev_main (the hot kernel).  Lane = placement, wave = 64 placements, every wave of a workgroup scores
// the same placements on different tokens, so a token's expert ids are wave-uniform:
//   * LDS holds, for the workgroup's placements and layer, the one-hot GPU mask of every expert
//     (tbl[e][p], uint32; zero for replicated experts), the replica info (FC, fallback) and
//     per-placement counters of the GPUs chosen for replicated experts.
//   * A wave loads 64 token-layers at once (one load per lane), packs the expert ids four per dword
//     and builds a per-token word with the replicated-slot mask, the anchor GPU and the replica
//     indices; the per-token loop broadcasts them with v_readlane, so the ids live in SGPRs.
//   * Per token-layer and lane: k conflict-free LDS reads (64 consecutive dwords per wave), OR of the
//     masks, then (rarely) the replicated slots, then two popcounts into per-lane accumulators.
#include <algorithm>

#include "eval_internal.h"

namespace tacg {
namespace {

constexpr int kMainThreads = 1024;
// About 32 workgroups of ev_main per CU: short enough that the last round leaves little idle time
// when the families' ragged last pieces make the workgroups uneven (measured 2 % faster than 4096
// on a Dirichlet family mix), long enough to amortise the table set-up and the flushes.
constexpr int64_t kTargetWorkgroups = 8192;

struct CountSegs {  // end token of every family
  uint32_t end[TACG_MAX_FAMILIES];
};

// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void zero_accumulators(const EvBase& a) {  // grid-stride
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const EvWs& w = a.ws;
  for (int64_t j = i; j < static_cast<int64_t>(a.L) * a.E; j += stride) w.cnt[j] = 0;
  for (int64_t j = i; j < static_cast<int64_t>(a.L) * 8; j += stride) w.flagbits[j] = 0;
  for (int64_t j = i; j < a.P; j += stride) {
    w.acc_home[j] = 0;
    w.acc_span[j] = 0;
  }
  for (int64_t j = i; j < static_cast<int64_t>(a.P) * a.F; j += stride) w.acc_fam[j] = 0;
  for (int64_t j = i; j < static_cast<int64_t>(even_up(a.P)) * a.L * a.G; j += stride) w.rep_load[j] = 0;
  if (i == 0) *w.n_bad = 0;
  for (int64_t j = i; j < bad_tile_words(a.N, a.L); j += stride) w.bad_tiles[j] = 0;
  if (a.stats) {
    for (int64_t j = i; j < static_cast<int64_t>(a.F) * a.L * a.E; j += stride) w.cnt_fam[j] = 0;
    for (int64_t j = i; j < static_cast<int64_t>(a.P) * a.F; j += stride) {
      w.acc_span_fam[j] = 0;
      w.acc_cross_fam[j] = 0;
      w.acc_hmass_fam[j] = 0;
    }
  }
}

__global__ __launch_bounds__(256) void ev_zero(EvBase a) { zero_accumulators(a); }

// Trace validation and dispatch counts: every token-layer's ids, read once.  A workgroup takes a contiguous range of the
// flattened trace (x = l * N + t) and walks the layers (with statistics: the families of the layers) it crosses,
// counting the dispatches of every expert in LDS.  A token-layer with an id out of range or a repeated id is flagged,
// counted (n_bad), left out of the counts, and marks its group of 64 consecutive token-layers in bad_tiles, so that
// ev_main checks the ids itself only in the few tiles that meet a marked group (the other two passes check every token when any
// is invalid).
// Bound by the read of the trace: the LDS adds of the counts hide behind it (2^19 tokens x 58 layers, top-8: 78 us
// without them, and 100 us with them, while they cost the trace pass of few placements a fifth of its time).
template <int K>
__global__ __launch_bounds__(256) void ev_valid(EvBase a, CountSegs segs) {
  __shared__ uint32_t ecnt[TACG_MAX_EXPERTS];
  const int64_t total = a.N * a.L;
  const int tid = threadIdx.x, lane = tid & 63;
  int64_t pos = total * blockIdx.x / gridDim.x;
  const int64_t end = total * (blockIdx.x + 1) / gridDim.x;
  const uint32_t E = static_cast<uint32_t>(a.E);
  uint32_t err = 0;
  for (int e = tid; e < a.E; e += blockDim.x) ecnt[e] = 0;
  __syncthreads();
  // the families' ends, one per lane: a segment's family is the number of ends at or before its first token
  static_assert(TACG_MAX_FAMILIES == 64, "a family per lane");
  const uint32_t fam_end = a.stats ? segs.end[lane] : 0u;
  int64_t l = pos / a.N, layer0 = l * a.N;  // layer of pos, and its first token-layer
  while (pos < end) {
    if (pos - layer0 >= a.N) {
      ++l;
      layer0 += a.N;
    }
    int f = 0;
    int64_t stop = min(end, layer0 + a.N);
    if (a.stats) {
      f = __popcll(__ballot(static_cast<int64_t>(fam_end) <= pos - layer0));
      stop = min(end, layer0 + static_cast<uint32_t>(__builtin_amdgcn_readlane(fam_end, f)));
    }
    const int64_t last = stop - 1;
    constexpr int kAhead = 2;  // steps in flight behind the current one
    TraceIds<K> ring[kAhead];
#pragma unroll
    for (int d = 0; d < kAhead; ++d) ring[d].fetch(a.trace + min(pos + tid + d * 256, last) * K);
    for (int64_t xb = pos; xb < stop; xb += kAhead * 256) {
#pragma unroll
      for (int d = 0; d < kAhead; ++d) {
        if (d > 0 && xb + d * 256 >= stop) break;  // a short segment: no step for its end
        const int64_t x = xb + d * 256 + tid;
        uint32_t raw[K];
        ring[d].unpack(raw);
        ring[d].fetch(a.trace + min(x + kAhead * 256, last) * K);
        const bool in = x < stop;
        bool ok = true, dup = false;
#pragma unroll
        for (int s = 0; s < K; ++s) {
          ok &= raw[s] < E;
#pragma unroll
          for (int q = 0; q < s; ++q) dup |= raw[s] == raw[q];
        }
        if (in && ok && !dup) {
#pragma unroll
          for (int s = 0; s < K; ++s)
            __hip_atomic_fetch_add(&ecnt[raw[s]], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        const bool bad = in && (!ok || dup);
        if (bad) {
          err |= (ok ? 0u : TACG_ERR_ID_RANGE) | (dup ? TACG_ERR_ID_DUP : 0u);
          atomicOr(&a.ws.bad_tiles[x >> 11], 1u << ((x >> 6) & 31));
        }
        const uint64_t b = __ballot(bad);
        if (b != 0u && lane == 0) atomicAdd(a.ws.n_bad, static_cast<unsigned long long>(__popcll(b)));
      }
    }
    barrier_after_lds_atomics();
    for (int e = tid; e < a.E; e += blockDim.x) {
      const uint32_t c = ecnt[e];
      if (c) {
        atomicAdd(&a.ws.cnt[l * a.E + e], c);
        if (a.stats) atomicAdd(&a.ws.cnt_fam[(static_cast<int64_t>(f) * a.L + l) * a.E + e], c);
      }
      ecnt[e] = 0;
    }
    __syncthreads();
    pos = stop;
  }
  if (err) atomicOr(a.d_err, err);
}

// Table validation and the replicated-expert marks.  Flat grid-stride loop over (p, l, e), four experts of a thread
// in flight (bound by the latency of the byte loads otherwise: 95 us at 1024 placements x 58 layers x 256 experts with three
// secondaries, 61 us with four).
constexpr int kFlagsAhead = 4;

// One expert's tables: error bits, and whether it has a (valid) secondary.
template <int R>
__device__ __forceinline__ bool has_secondary(uint8_t g0, const uint8_t* sec, int G, uint32_t& err) {
  if (g0 >= G) err |= TACG_ERR_TABLE;
  bool any = false;
  uint32_t seen = g0 < G ? (1u << g0) : 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint8_t g = sec[r];
    if (g == kNone) continue;
    if (g >= G || (seen >> g) & 1u) {
      err |= TACG_ERR_TABLE;
      continue;
    }
    seen |= 1u << g;
    any = true;
  }
  return any;
}

template <int R>
__global__ __launch_bounds__(256) void ev_flags(EvBase a) {
  const int64_t n = static_cast<int64_t>(a.P) * a.L * a.E;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  uint32_t err = 0;
  for (int64_t pe0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; pe0 < n; pe0 += kFlagsAhead * stride) {
    uint8_t prim[kFlagsAhead], sec[kFlagsAhead][R > 0 ? R : 1];
#pragma unroll
    for (int u = 0; u < kFlagsAhead; ++u) {
      const int64_t pe = min(pe0 + u * stride, n - 1);
      prim[u] = a.primary[pe];
#pragma unroll
      for (int r = 0; r < R; ++r) sec[u][r] = a.secondary[pe * R + r];
    }
#pragma unroll
    for (int u = 0; u < kFlagsAhead; ++u) {
      const int64_t pe = pe0 + u * stride;
      if (pe >= n) break;
      if (has_secondary<R>(prim[u], sec[u], a.G, err)) {
        // every placement marks the same few experts: set a bit only when a device-scope read does
        // not show it yet (a stale read costs one extra atomic, never a missing bit)
        const int e = static_cast<int>(pe % a.E);
        const int l = static_cast<int>((pe / a.E) % a.L);
        uint32_t* w = &a.ws.flagbits[l * 8 + (e >> 5)];
        const uint32_t bit = 1u << (e & 31);
        if (!(__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) atomicOr(w, bit);
      }
    }
  }
  if (err) atomicOr(a.d_err, err);
}

// Compact indices of the marked experts of layer l (256 threads, one per expert), also into LDS.
struct RepList {
  int32_t cnt;
  int32_t expert[TACG_MAX_REPLICATED];
};

__device__ __forceinline__ void list_replicated(const EvBase& a, int l, const uint32_t* bits, RepList& list) {
  const int e = threadIdx.x;
  int32_t& cnt = list.cnt;
  if (e == 0) cnt = 0;
  __syncthreads();
  if (e < a.E) {
    const bool mark = (bits[e >> 5] >> (e & 31)) & 1u;
    // rank among marked experts = number of marked experts below e
    int rank = 0;
    for (int q = 0; q < (e >> 5); ++q) rank += __popc(bits[q]);
    rank += __popc(bits[e >> 5] & ((1u << (e & 31)) - 1u));
    uint8_t r = kNone;
    if (mark) {
      atomicAdd(&cnt, 1);
      if (rank < TACG_MAX_REPLICATED) {
        r = static_cast<uint8_t>(rank);
        a.ws.rep_list[l * TACG_MAX_REPLICATED + rank] = e;
        list.expert[rank] = e;
      }
    }
    a.ws.rep_of[static_cast<int64_t>(l) * a.E + e] = r;
  }
  barrier_after_lds_atomics();
  if (e == 0) {
    a.ws.n_rep[l] = min(cnt, TACG_MAX_REPLICATED);
    if (cnt > TACG_MAX_REPLICATED) atomicOr(a.d_err, TACG_ERR_LIMIT);
  }
}

__global__ __launch_bounds__(256) void ev_replist(EvBase a) {  // grid (L)
  __shared__ RepList list;
  list_replicated(a, blockIdx.x, a.ws.flagbits + blockIdx.x * 8, list);
}

// Feasible candidates and fallback for every (placement, layer, replicated expert).  A wave takes four placements of a
// layer, sixteen lanes each: the lanes first hold the placement's loads (two GPUs per lane) for the guard, then one replicated
// expert each.  grid (ceil(P / 16), L), 256 threads.  Bound by latency: one thread per placement working through its sixteen
// experts took 34 us for two placements and 44 us for 1024 (58 layers, 32 GPUs, 16 experts with three secondaries); this takes
// 5 and 19 us.
typedef int64_t RepLoads[16][TACG_MAX_GPUS];

__device__ __forceinline__ void candidates_of(const EvBase& a, int l, int block, int nrep, const int32_t* experts,
                                              RepLoads& loads) {
  static_assert(TACG_MAX_REPLICATED == 16 && TACG_MAX_GPUS == 32, "sixteen lanes per placement");
  const int lane = threadIdx.x & 63, i16 = lane & 15, local = threadIdx.x >> 4;
  const int p = block * 16 + local, pc = min(p, a.P - 1);
  const int G = a.G;
  const int64_t* ref = a.load_ref + (static_cast<int64_t>(pc) * a.L + l) * G;
  int64_t v[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = i16 + 16 * j;
    v[j] = m < G ? ref[min(m, G - 1)] : 0;
    loads[local][m] = v[j];
  }
  // this lane's expert: its candidate set
  uint32_t cand = 0;
  if (i16 < nrep) {
    const int e = experts[i16];
    const int64_t pe = (static_cast<int64_t>(pc) * a.L + l) * a.E + e;
    const uint8_t g0 = a.primary[pe];
    if (g0 < G) cand |= 1u << g0;
    for (int q = 0; q < a.R; ++q) {
      const uint8_t g = a.secondary[pe * a.R + q];
      if (g < G) cand |= 1u << g;
    }
  }
  // eq. feasible-set with the mean load of eq. mean-load, exact in 128-bit integers
  uint32_t feas = (G == 32) ? 0xffffffffu : ((1u << G) - 1u);
  if (a.theta_den != 0) {
    // the total as sums of the 32-bit halves over the sixteen lanes
    int64_t hi = (v[0] >> 32) + (v[1] >> 32);
    int64_t lo = (v[0] & 0xffffffffll) + (v[1] & 0xffffffffll);
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) {
      hi += __shfl_xor(hi, o, 64);
      lo += __shfl_xor(lo, o, 64);
    }
    const __int128 total = static_cast<__int128>(hi) * (int64_t(1) << 32) + lo;
    const __int128 rhs = static_cast<__int128>(a.theta_den + a.theta_num) * total;
    feas = 0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bool ok = i16 + 16 * j < G && static_cast<__int128>(a.theta_den) * G * v[j] <= rhs;
      const uint64_t bal = __ballot(ok);
      feas |= (static_cast<uint32_t>(bal >> (lane & 48)) & 0xffffu) << (16 * j);
    }
  }
  if (p >= a.P || i16 >= nrep) return;
  // the loads were staged by lanes of this wave: the LDS keeps its operations in order
  __asm__ __volatile__("" ::: "memory");
  if (cand == 0) cand = 1u;  // invalid table (already flagged): keep the choice in range
  uint32_t fc = cand & feas;
  if (fc == 0) fc = cand;
  // least-loaded feasible candidate, ties to the lowest GPU
  int best = __builtin_ctz(fc);
  int64_t bestv = loads[local][best];
  for (uint32_t rest = fc & (fc - 1u); rest != 0u; rest &= rest - 1u) {
    const int m = __builtin_ctz(rest);
    const int64_t x = loads[local][m];
    if (x < bestv) {
      best = m;
      bestv = x;
    }
  }
  // bit 31: the expert has a single candidate in this placement (it is served by its primary and
  // belongs to the GPUs the token reaches before any multi-candidate slot is resolved)
  const uint32_t single = (__popc(cand) == 1) ? 0x80000000u : 0u;
  a.ws.rep_info[(static_cast<int64_t>(l) * TACG_MAX_REPLICATED + i16) * a.P + p] =
      make_uint2(fc, static_cast<uint32_t>(best) | single);
}

__global__ __launch_bounds__(256) void ev_repinfo(EvBase a) {
  __shared__ RepLoads loads;
  const int l = blockIdx.y, nrep = a.ws.n_rep[l];
  if (nrep > 0) candidates_of(a, l, blockIdx.x, nrep, a.ws.rep_list + l * TACG_MAX_REPLICATED, loads);
}

// ev_zero, ev_flags, ev_replist and ev_repinfo in one launch, a workgroup per layer: all but the clearing is per layer.
// For short tables only, where four launches cost more than the passes: a workgroup takes kPrepTables entries per layer about
// as long as they do, and with secondaries kPrepPlace placements, whose candidate sets it works through sixteen at a time.
// Whole scoring calls, four launches / one, at 12 layers x 1000 tokens, top-2: E = 128 without secondaries 23.2 / 20.4 us
// at 8 placements, 25.3 / 25.1 at 32, 24.6 / 27.6 at 64; with 6 x 3 replicas 33.3 / 26.7, 37.3 / 37.6 and 38.0 / 48.9; E = 16 with
// 6 x 3 replicas 32.3 / 25.0 at 16 (E = 8), 38.5 / 40.0 at 128, 71 / 103 at 512.  grid (L), 256 threads.
constexpr int64_t kPrepTables = 4096, kPrepPlace = 64;

template <int R>
__global__ __launch_bounds__(256) void ev_prep(EvBase a) {
  __shared__ uint32_t bits[8];
  __shared__ RepList list;
  __shared__ RepLoads loads;
  const int l = blockIdx.x, tid = threadIdx.x;
  zero_accumulators(a);
  if (tid < 8) bits[tid] = 0;
  __syncthreads();
  uint32_t err = 0;
  for (int i = tid; i < a.P * a.E; i += 256) {
    const int p = i / a.E, e = i - p * a.E;
    const int64_t pe = (static_cast<int64_t>(p) * a.L + l) * a.E + e;
    uint8_t sec[R > 0 ? R : 1];
#pragma unroll
    for (int r = 0; r < R; ++r) sec[r] = a.secondary[pe * R + r];
    if (has_secondary<R>(a.primary[pe], sec, a.G, err)) atomicOr(&bits[e >> 5], 1u << (e & 31));
  }
  barrier_after_lds_atomics();
  list_replicated(a, l, bits, list);
  __syncthreads();
  const int nrep = min(list.cnt, TACG_MAX_REPLICATED);
  if (R > 0 && nrep > 0)
    for (int b = 0; b * 16 < a.P; ++b) candidates_of(a, l, b, nrep, list.expert, loads);
  if (err) atomicOr(a.d_err, err);
}

// ------------------------------------------------------------------------------------------------
// The trace pass.  PPL placements per lane (one 8- or 16-byte LDS read per slot serves all of them);
// a workgroup scores 64 * PPL placements of one layer on one piece of one family's tokens.
// grid (placement blocks, pieces, L).  ev_valid has already checked the ids, and only tiles it marked check them
// again, to leave their invalid token-layers out.
// Choices for replicated experts are counted in 16-bit LDS counters (two per dword).  After every
// round of at most 65535 / K tokens (so that they cannot overflow) each thread adds a fixed set of
// them into 32-bit registers and clears them; the registers go to the workspace once per workgroup.
//
// Per-token word `info` built by the lane that loaded the token-layer (wave-uniform after v_readlane):
//   K <= 8:  bits 0-7 replicated-slot mask, 8-12 band position of the anchor GPU within its family's
//            band, then 4-bit replica indices of the first four replicated slots (13-16 ... 25-28);
//   K > 8:   bits 0-15 replicated-slot mask, 16-20 band position, replica indices of the first two
//            replicated slots (21-24, 25-28).
// Further replicated slots of a token look their index up in LDS.
template <int K>
struct InfoLayout {
  static constexpr int kMaskBits = K <= 8 ? 8 : 16;
  static constexpr int kHomeShift = kMaskBits;
  static constexpr int kRepShift = kMaskBits + 5;
  static constexpr int kRepSlots = K <= 8 ? 4 : 2;
  static constexpr uint32_t kBad = 1u << 31;  // the token-layer is not scored (invalid ids)
};

// Index of the lowest set bit, 0xffffffff for 0 (the hardware v_ffbl_b32 result).
__device__ __forceinline__ uint32_t find_first_bit(uint32_t x) {
  uint32_t r;
  asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

template <int K, int PPL, bool NARROW, bool STATS>
struct Scorer {
  static constexpr int PW = 64 * PPL;
  static constexpr int KB = (K + 3) / 4;  // dwords of 8-bit expert ids per token-layer
  static constexpr int kRowShift = PPL == 2 ? 9 : 10;  // log2 of a table row in bytes (PW * 4)
  using IL = InfoLayout<K>;

  const char* tbl_lane;   // LDS table base + this lane's column offset
  uint32_t row_bytes;     // PW * 4, held in a VGPR
  const uint2* rinfo;     // [MAX_REP][PW]
  uint32_t* rcnt;         // [G][PW / 2]
  const uint8_t* rep_of;  // [E]
  int lane;
  uint32_t acc_span[PPL], acc_home[PPL];

  // one-hot GPU masks of the token's single-candidate experts, OR-ed per placement
  __device__ __forceinline__ void gather(const uint32_t (&ids)[KB], uint32_t (&m)[PPL]) const {
#pragma unroll
    for (int q = 0; q < PPL; ++q) m[q] = 0;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const uint32_t id = __builtin_amdgcn_ubfe(ids[s >> 2], 8 * (s & 3), 8);
      // row stride in an opaque VGPR: one scalar extract and one v_mad_u32_u24 per slot (left to
      // itself the compiler moves the shift into two scalar instructions for half of the slots)
      const char* base = tbl_lane + __umul24(id, row_bytes);
      if constexpr (PPL == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(base);
        m[0] |= v.x;
        m[1] |= v.y;
      } else {
        const uint4 v = *reinterpret_cast<const uint4*>(base);
        m[0] |= v.x;
        m[1] |= v.y;
        m[2] |= v.z;
        m[3] |= v.w;
      }
    }
  }

  // Replicated slots in slot order: the lowest-numbered feasible candidate the token already
  // reaches, else the anchor if it is a feasible candidate, else the least-loaded feasible candidate.
  // rinfo[r][p] = (FC mask, packed fallbacks): byte i holds 32 + (the choice when no candidate is
  // reached) for the anchor at band position i (bands of up to 4 GPUs; wider bands keep 32 + the
  // least-loaded feasible candidate and test the anchor here).  ffbl(0) = 0xffffffff, so min(ffbl(x), 32 + fb)
  // selects the reached candidate when there is one; the shift and the counter row use its low 5 bits.
  __device__ __forceinline__ void resolve(uint32_t info, const uint32_t (&ids)[KB], uint32_t (&m)[PPL]) {
    const uint32_t repmask = info & ((1u << IL::kMaskBits) - 1u);
    if (!repmask) return;
    const uint32_t hshift = 8u * ((info >> IL::kHomeShift) & 31u);  // 8 * band position of the anchor
    // a scalar loop over the set bits of the (wave-uniform) mask: the replicated slots only
    int nth = 0;
    for (uint32_t rem = repmask; rem != 0u; rem &= rem - 1u, ++nth) {
      const int s = __builtin_ctz(rem);
      uint32_t r;
      if (nth < IL::kRepSlots) {
        r = (info >> (IL::kRepShift + 4 * nth)) & 15u;
      } else {
        r = rep_of[__builtin_amdgcn_ubfe(ids[s >> 2], 8 * (s & 3), 8)];
      }
      const uint2* rp = rinfo + r * PW + lane * PPL;
      uint2 ri[PPL];
#pragma unroll
      for (int q = 0; q < PPL; q += 2) {
        const uint4 v = *reinterpret_cast<const uint4*>(rp + q);
        ri[q] = make_uint2(v.x, v.y);
        ri[q + 1] = make_uint2(v.z, v.w);
      }
#pragma unroll
      for (int q = 0; q < PPL; ++q) {
        const uint32_t x = ri[q].x & m[q];
        uint32_t fb;
        if constexpr (NARROW) {
          fb = __builtin_amdgcn_ubfe(ri[q].y, hshift, 8);
        } else {
          const uint32_t h = home_start + (hshift >> 3);
          fb = ((ri[q].x >> h) & 1u) ? 32u + h : ri[q].y;
        }
        const uint32_t pick = min(find_first_bit(x), fb) & 31u;
        m[q] |= 1u << pick;
        __hip_atomic_fetch_add(&rcnt[(pick * PW + lane * PPL + q) >> 1], 1u << (16 * (q & 1)), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }

  uint32_t home_start;
  uint32_t band_starts;     // STATS: bit b set when a family band starts at GPU b
  uint32_t acc_cross[PPL];  // STATS: token-layers whose cards span more than one band

  __device__ __forceinline__ void account(uint32_t info, const uint32_t (&m)[PPL]) {
    const uint32_t not_h = ~(1u << (home_start + ((info >> IL::kHomeShift) & 31u)));
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      acc_span[q] += __popc(m[q]);
      acc_home[q] += __popc(m[q] & not_h);
      if constexpr (STATS) {
        // The bands are intervals that tile the GPUs, so the cards lie in more than one band exactly
        // when a band starts in (lowest card, highest card].  With lo / hi the lowest / highest card,
        // (2 << hi) - (2 << lo) (mod 2^32, so hi = 31 works) has exactly those bits set.
        // (m == 0 only after a flagged table error; the masks keep every shift defined)
        const uint32_t lo = find_first_bit(m[q]) & 31u;
        const uint32_t top = 0x80000000u >> (__clz(static_cast<int>(m[q])) & 31);  // 1 << hi
        const uint32_t range = (top << 1) + (0xfffffffeu << lo);
        acc_cross[q] += (band_starts & range) != 0u ? 1u : 0u;
      }
    }
  }
};

// Token loop of one workgroup (see ev_main).  NARROW: the family's band has at most 4 GPUs, so the
// fallback choices are packed per band position.
template <int K, int PPL, bool NARROW, bool STATS, bool CHECK>
__device__ __forceinline__ void score_piece(const EvArgs& a, const uint32_t* tbl, const uint2* rinfo, uint32_t* rcnt,
                                            const uint8_t* rep_of, int l, int p0, int nrep, uint32_t t_begin, uint32_t t_end, uint32_t off_f,
                                            uint32_t hs, uint32_t hz, int f,
                                            uint32_t (&acc_span)[PPL], uint32_t (&acc_home)[PPL],
                                            uint32_t (&acc_cross)[PPL], uint32_t& n_scored) {
  using S = Scorer<K, PPL, NARROW, STATS>;
  using IL = InfoLayout<K>;
  constexpr int PW = S::PW;
  constexpr int KB = S::KB;
  constexpr int U = 4;             // token-layers scored together (independent LDS reads in flight)
  constexpr uint32_t round_tokens = 65535u / K;
  // each thread folds the same 2 * kRcntPerThread 16-bit counters after every round
  constexpr int kRcntPerThread = (TACG_MAX_GPUS * PW / 2 + kMainThreads - 1) / kMainThreads;
  uint32_t rsum[2 * kRcntPerThread];
#pragma unroll
  for (int c = 0; c < 2 * kRcntPerThread; ++c) rsum[c] = 0;
  const int E = a.E, G = a.G, L = a.L;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwaves = blockDim.x >> 6;
  // Tokens are counted from the piece's first, at most 2^26 of them, so that no step past its end wraps at the last
  // tokens of a trace of nearly 2^32 (top-1).
  const int16_t* trace_p = a.trace + (static_cast<int64_t>(l) * a.N + t_begin) * K;
  const uint32_t n_piece = t_end - t_begin, pos0 = t_begin - off_f;  // pos0: the piece's position in its family
  S sc;
  sc.tbl_lane = reinterpret_cast<const char*>(tbl) + lane * PPL * 4;
  asm volatile("v_mov_b32 %0, %1" : "=v"(sc.row_bytes) : "i"(S::PW * 4));
  sc.rinfo = rinfo;
  sc.rcnt = rcnt;
  sc.rep_of = rep_of;
  sc.lane = lane;
  sc.home_start = hs;
  sc.band_starts = a.band_starts;
#pragma unroll
  for (int q = 0; q < PPL; ++q) sc.acc_span[q] = sc.acc_home[q] = sc.acc_cross[q] = 0;

  for (uint32_t r_begin = 0; r_begin < n_piece; r_begin += round_tokens) {
    const uint32_t r_end = min(n_piece, r_begin + round_tokens);
    for (uint32_t tile = r_begin + wave * 64u; tile < r_end; tile += nwaves * 64u) {
      // ---- per-lane preprocessing of token-layer (tile + lane) ----
      const uint32_t t = tile + lane;
      uint32_t pk[KB];
#pragma unroll
      for (int w = 0; w < KB; ++w) pk[w] = 0;
      // does the tile meet a group of 64 flattened token-layers that ev_valid marked? (wave-uniform;
      // only the variant for traces with an invalid token-layer reads the marks)
      bool marked = false;
      if constexpr (CHECK) {
        const int64_t x0 = static_cast<int64_t>(l) * a.N + t_begin + tile;
        const int64_t g0 = x0 >> 6, g1 = min(x0 + 63, static_cast<int64_t>(L) * a.N - 1) >> 6;
        marked = (((a.ws.bad_tiles[g0 >> 5] >> (g0 & 31)) | (a.ws.bad_tiles[g1 >> 5] >> (g1 & 31))) & 1u) != 0u;
      }
      uint32_t info = 0;
      bool bad = false;
      if (t < r_end) {
        const int16_t* idp = trace_p + static_cast<int64_t>(t) * K;
        uint32_t raw[K];
#pragma unroll
        for (int s = 0; s < K; ++s) raw[s] = static_cast<uint16_t>(idp[s]);
        int nth = 0;
#pragma unroll
        for (int s = 0; s < K; ++s) {
          const uint32_t id = min(raw[s], static_cast<uint32_t>(E - 1));
          const uint32_t r = rep_of[id];
          if (r != kNone) {
            info |= 1u << s;
            if (nth < IL::kRepSlots) info |= r << (IL::kRepShift + 4 * nth);
            ++nth;
          }
          pk[s >> 2] |= id << (8 * (s & 3));
        }
        info |= ((pos0 + t) % hz) << IL::kHomeShift;
        if (marked) {
          // an invalid token-layer (flagged by ev_valid) is not scored; its ids stay clamped in
          // range, unused
          bool ok = true, dup = false;
#pragma unroll
          for (int s = 0; s < K; ++s) {
            ok &= raw[s] < static_cast<uint32_t>(E);
#pragma unroll
            for (int q = 0; q < s; ++q) dup |= raw[s] == raw[q];
          }
          bad = !ok || dup;
          if (bad) info = IL::kBad;
        }
      }
      const uint32_t ntile = min(64u, r_end - tile);
      const uint32_t nbad = static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(bad)));
      n_scored += ntile - nbad;
      uint32_t j = 0;
      if (nbad == 0u) {  // wave-uniform: a tile with invalid token-layers takes the loop below
        for (; j + U <= ntile; j += U) {
          uint32_t ids[U][KB], tinfo[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int w = 0; w < KB; ++w) ids[u][w] = __builtin_amdgcn_readlane(pk[w], j + u);
            tinfo[u] = __builtin_amdgcn_readlane(info, j + u);
          }
          uint32_t m[U][PPL];
#pragma unroll
          for (int u = 0; u < U; ++u) sc.gather(ids[u], m[u]);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            sc.resolve(tinfo[u], ids[u], m[u]);
            sc.account(tinfo[u], m[u]);
          }
        }
      }
      // the tile's last token-layers, or all of a tile with invalid ones, one at a time
      for (; j < ntile; ++j) {
        uint32_t ids[KB];
#pragma unroll
        for (int w = 0; w < KB; ++w) ids[w] = __builtin_amdgcn_readlane(pk[w], j);
        const uint32_t tinfo = __builtin_amdgcn_readlane(info, j);
        if (tinfo & IL::kBad) continue;
        uint32_t m[PPL];
        sc.gather(ids, m);
        sc.resolve(tinfo, ids, m);
        sc.account(tinfo, m);
      }
    }
    if (nrep > 0) {  // fold the 16-bit choice counters of this round into registers (nrep is workgroup-uniform)
      barrier_after_lds_atomics();
#pragma unroll
      for (int c = 0; c < kRcntPerThread; ++c) {
        const int i = threadIdx.x + c * kMainThreads;
        if (i < G * PW / 2) {
          const uint32_t v = rcnt[i];
          rsum[2 * c] += v & 0xffffu;
          rsum[2 * c + 1] += v >> 16;
          rcnt[i] = 0;
        }
      }
      __syncthreads();
    }
  }
  if (nrep > 0) {  // one global add per counter and workgroup
#pragma unroll
    for (int c = 0; c < kRcntPerThread; ++c) {
      const int i = threadIdx.x + c * kMainThreads;
      if (i < G * PW / 2) {
        const int g = (2 * i) / PW, q = 2 * i - g * PW, p = p0 + q;  // p even
        // placements p and p + 1 are adjacent: one 64-bit add carries both counts (each below 2^32,
        // so nothing carries from the low half); a slot past P is padding
        const uint64_t pair = static_cast<uint64_t>(rsum[2 * c]) | (static_cast<uint64_t>(rsum[2 * c + 1]) << 32);
        unsigned long long* dst = reinterpret_cast<unsigned long long*>(
            a.ws.rep_load + (static_cast<int64_t>(l) * G + g) * even_up(a.P) + p);
        if (p < a.P && pair) atomicAdd(dst, static_cast<unsigned long long>(pair));
        if constexpr (STATS) {  // replicated-slot dispatches served inside the family's own band
          if (static_cast<uint32_t>(g) - hs < hz) {
            unsigned long long* hm = a.ws.acc_hmass_fam + static_cast<int64_t>(f) * a.P + p;
            if (p < a.P && rsum[2 * c]) atomicAdd(hm, static_cast<unsigned long long>(rsum[2 * c]));
            if (p + 1 < a.P && rsum[2 * c + 1]) atomicAdd(hm + 1, static_cast<unsigned long long>(rsum[2 * c + 1]));
          }
        }
      }
    }
  }

#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    acc_span[q] = sc.acc_span[q];
    acc_home[q] = sc.acc_home[q];
    acc_cross[q] = sc.acc_cross[q];
  }
}

template <int K, int PPL, bool STATS>
__global__ __launch_bounds__(kMainThreads) void ev_main(EvArgs a) {
  extern __shared__ __align__(16) uint32_t lds[];
  constexpr int PW = 64 * PPL;
  const int E = a.E, G = a.G, L = a.L;
  // XCD-aware order: the hardware hands workgroup b to XCD b mod 8, so each XCD takes a contiguous
  // run of virtual ids v, in which the placement blocks of one (piece, layer) tile are adjacent.
  // They run together on that XCD and share its L2 for the tile's trace rows.
  const uint32_t total = gridDim.x, b = blockIdx.x;
  const uint32_t xcd = b % kXcds, per = total / kXcds, rem = total % kXcds;
  const uint32_t v = xcd * per + min(xcd, rem) + b / kXcds;
  const int npb = a.n_pblocks;
  const int pb = static_cast<int>(v % npb);
  const int tile = static_cast<int>(v / npb);
  const int piece = tile % a.n_pieces, l = tile / a.n_pieces;
  const int p0 = pb * PW;
  const int nrep = a.ws.n_rep[l];
  uint32_t* tbl = lds;                                                // [E][PW] one-hot GPU masks
  uint2* rinfo = reinterpret_cast<uint2*>(lds + E * PW);              // [MAX_REP][PW] (FC, fallback)
  uint32_t* rcnt = lds + E * PW + 2 * TACG_MAX_REPLICATED * PW;       // [G][PW / 2] two u16 counters
  uint8_t* rep_of = reinterpret_cast<uint8_t*>(rcnt + G * PW / 2);    // [E]
  // [kRed][PW] per-placement cost sums of the workgroup's waves, then the sum of their n_scored
  constexpr int kRed = STATS ? 3 : 2;  // span, home (and cross)
  uint32_t* red = reinterpret_cast<uint32_t*>(rep_of + ((E + 255) & ~255));  // rep_of padded to 256 bytes
  const uint8_t* rep_of_g = a.ws.rep_of + static_cast<int64_t>(l) * E;

  // one-hot primary GPU of every expert that has a single candidate in the placement; zero for the
  // multi-candidate ones (they are resolved per token)
  for (int i = threadIdx.x; i < E * PW; i += blockDim.x) {
    const int e = i / PW, q = i - e * PW, p = p0 + q;
    uint32_t v = 0;
    if (p < a.P) {
      const uint8_t r = rep_of_g[e];
      const bool single = (r == kNone) ||
          (a.ws.rep_info[(static_cast<int64_t>(l) * TACG_MAX_REPLICATED + r) * a.P + p].y >> 31);
      if (single) {
        const uint8_t g = a.primary[(static_cast<int64_t>(p) * L + l) * E + e];
        v = g < G ? (1u << g) : 0u;
      }
    }
    tbl[i] = v;
  }
  const uint4 pc = a.piece[piece];
  const uint32_t t_begin = pc.x, t_end = pc.y, off_f = pc.z;
  const uint32_t hs = pc.w & 0xffu, hz = (pc.w >> 8) & 0xffu;
  const int f = static_cast<int>(pc.w >> 16);
  {
    for (int i = threadIdx.x; i < nrep * PW; i += blockDim.x) {
      const int r = i / PW, q = i - r * PW, p = p0 + q;
      uint2 v = make_uint2(1u, 0u);
      if (p < a.P) v = a.ws.rep_info[(static_cast<int64_t>(l) * TACG_MAX_REPLICATED + r) * a.P + p];
      v.y &= 31u;
      uint32_t pack = 32u + v.y;  // bands wider than 4 GPUs: the plain fallback (+32)
      if (hz <= 4) {
        pack = 0;
        for (uint32_t b = 0; b < hz; ++b) {
          const uint32_t h = hs + b;
          pack |= (32u + (((v.x >> h) & 1u) ? h : v.y)) << (8 * b);
        }
      }
      rinfo[i] = make_uint2(v.x, pack);
    }
  }
  for (int i = threadIdx.x; i < G * PW / 2; i += blockDim.x) rcnt[i] = 0;
  for (int i = threadIdx.x; i < kRed * PW + 1; i += blockDim.x) red[i] = 0;
  for (int i = threadIdx.x; i < E; i += blockDim.x) rep_of[i] = rep_of_g[i];
  __syncthreads();

  const int lane = threadIdx.x & 63;
  // ev_valid counted the invalid token-layers: almost always none, and then no tile checks its ids
  const bool any_bad = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(*a.ws.n_bad != 0u)) != 0u;

  uint32_t acc_span[PPL], acc_home[PPL], acc_cross[PPL];
  uint32_t n_scored = 0;  // token-layers scored by this wave
  if (any_bad) {  // a trace with invalid token-layers: the variant that checks the marked tiles
    if (hz <= 4) {
      score_piece<K, PPL, true, STATS, true>(a, tbl, rinfo, rcnt, rep_of, l, p0, nrep, t_begin, t_end,
                                             off_f, hs, hz, f, acc_span, acc_home, acc_cross, n_scored);
    } else {
      score_piece<K, PPL, false, STATS, true>(a, tbl, rinfo, rcnt, rep_of, l, p0, nrep, t_begin, t_end,
                                              off_f, hs, hz, f, acc_span, acc_home, acc_cross, n_scored);
    }
  } else if (hz <= 4) {
    score_piece<K, PPL, true, STATS, false>(a, tbl, rinfo, rcnt, rep_of, l, p0, nrep, t_begin, t_end,
                                            off_f, hs, hz, f, acc_span, acc_home, acc_cross, n_scored);
  } else {
    score_piece<K, PPL, false, STATS, false>(a, tbl, rinfo, rcnt, rep_of, l, p0, nrep, t_begin, t_end,
                                             off_f, hs, hz, f, acc_span, acc_home, acc_cross, n_scored);
  }

  // ---- flush: each wave adds its per-placement costs into the workgroup's LDS sums as it finishes;
  // then one global add per placement and accumulator, contiguous in p ----
#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    const int c = lane * PPL + q;
    __hip_atomic_fetch_add(&red[c], acc_span[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_add(&red[PW + c], acc_home[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if constexpr (STATS)
      __hip_atomic_fetch_add(&red[2 * PW + c], acc_cross[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  if constexpr (STATS) {
    if (lane == 0) __hip_atomic_fetch_add(&red[kRed * PW], n_scored, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  barrier_after_lds_atomics();
  for (int c = threadIdx.x; c < PW; c += blockDim.x) {
    const int p = p0 + c;
    if (p < a.P) {
      const uint32_t span = red[c], home = red[PW + c];
      if (span) atomicAdd(&a.ws.acc_span[p], static_cast<unsigned long long>(span));
      if (home) {
        atomicAdd(&a.ws.acc_home[p], static_cast<unsigned long long>(home));
        atomicAdd(&a.ws.acc_fam[static_cast<int64_t>(f) * a.P + p], static_cast<unsigned long long>(home));
      }
      if constexpr (STATS) {
        // |cards| - 1 summed over the workgroup's token-layers (each has at least one card)
        const int64_t fp = static_cast<int64_t>(f) * a.P + p;
        const uint32_t sp = span - red[kRed * PW];
        if (sp) atomicAdd(&a.ws.acc_span_fam[fp], static_cast<unsigned long long>(sp));
        if (red[2 * PW + c]) atomicAdd(&a.ws.acc_cross_fam[fp], static_cast<unsigned long long>(red[2 * PW + c]));
      }
    }
  }
}

// Loads and costs.  A workgroup takes one layer and `run` placements, a wave one placement at a time, as
// placement_load_kernel.  grid (ceil(P / run), L).
constexpr int kLoadWaves = 8;

__global__ __launch_bounds__(64 * kLoadWaves) void ev_finalize(EvBase a, int run, uint64_t* __restrict__ cost_home,
                                                               uint64_t* __restrict__ cost_span,
                                                               uint32_t* __restrict__ load,
                                                               uint64_t* __restrict__ cost_home_fam) {
  __shared__ uint32_t acc[kLoadWaves][TACG_MAX_GPUS];
  const int l = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int E = a.E, G = a.G, L = a.L;
  // dispatches of the experts that are served by their primary in every placement (a replicated one's are its choices)
  uint32_t d[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = lane + 64 * q;
    const int64_t le = static_cast<int64_t>(l) * E + min(e, E - 1);
    d[q] = e < E && a.ws.rep_of[le] == kNone ? a.ws.cnt[le] : 0u;
  }
  const int p1 = min(a.P, static_cast<int>(blockIdx.x + 1) * run);
  uint8_t next[4];
  uint32_t next_rep = 0;
  auto fetch = [&](int p) {
    const int pc = min(p, a.P - 1);
    const uint8_t* src = a.primary + (static_cast<int64_t>(pc) * L + l) * E;
#pragma unroll
    for (int q = 0; q < 4; ++q) next[q] = src[min(lane + 64 * q, E - 1)];
    next_rep = a.ws.rep_load[(static_cast<int64_t>(l) * G + min(lane, G - 1)) * even_up(a.P) + pc];
  };
  int p = blockIdx.x * run + wave;
  fetch(p);
  for (; p < p1; p += nw) {
    uint32_t g[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) g[q] = next[q];
    const uint32_t rep = next_rep;
    fetch(p + nw);
    if (lane < G) acc[wave][lane] = rep;
    __asm__ __volatile__("" ::: "memory");  // the LDS keeps a wave's operations in order
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (d[q] && g[q] < static_cast<uint32_t>(G))
        __hip_atomic_fetch_add(&acc[wave][g[q]], d[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __asm__ __volatile__("" ::: "memory");
    if (lane < G) load[(static_cast<int64_t>(p) * L + l) * G + lane] = acc[wave][lane];
    if (l == 0) {
      if (lane == 0) {
        cost_home[p] = a.ws.acc_home[p];
        // |cards| - 1 per scored token-layer (every scored token-layer has at least one card)
        cost_span[p] = a.ws.acc_span[p] - (static_cast<uint64_t>(a.N) * static_cast<uint64_t>(L) - *a.ws.n_bad);
      }
      if (cost_home_fam && lane < a.F)
        cost_home_fam[static_cast<int64_t>(p) * a.F + lane] = a.ws.acc_fam[static_cast<int64_t>(lane) * a.P + p];
    }
  }
}

// App. C statistics per (placement, family): home-family dispatch mass = dispatches of the family's
// tokens to single-candidate experts whose primary lies in the family's band (from the per-family
// dispatch counts) + replicated-slot choices inside the band (counted by the trace pass).
// grid (P, F), up to 1024 threads.
__global__ __launch_bounds__(1024) void ev_stats(EvArgs a, uint64_t* __restrict__ span_fam,
                                                uint64_t* __restrict__ cross_fam, uint64_t* __restrict__ hmass_fam) {
  __shared__ unsigned long long red[16];
  const int p = blockIdx.x, f = blockIdx.y;
  const int E = a.E, L = a.L;
  const uint4 r = a.band4[f >> 2];
  const uint32_t bw = (f & 3) == 0 ? r.x : (f & 3) == 1 ? r.y : (f & 3) == 2 ? r.z : r.w;
  const uint32_t hs = bw & 0xffu, hz = (bw >> 8) & 0xffu;
  unsigned long long s = 0;
  const int64_t n = static_cast<int64_t>(L) * E;
#pragma unroll 4
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {  // (l, e) flattened
    const uint32_t g = a.primary[static_cast<int64_t>(p) * n + i];
    const uint32_t c = a.ws.cnt_fam[static_cast<int64_t>(f) * n + i];
    s += (a.ws.rep_of[i] == kNone && g - hs < hz) ? c : 0u;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t pf = static_cast<int64_t>(p) * a.F + f, fp = static_cast<int64_t>(f) * a.P + p;
    unsigned long long t = 0;
    for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) t += red[w];
    hmass_fam[pf] = t + a.ws.acc_hmass_fam[fp];
    span_fam[pf] = a.ws.acc_span_fam[fp];
    cross_fam[pf] = a.ws.acc_cross_fam[fp];
  }
}

template <int K, int PPL, bool STATS>
int launch_main(const EvArgs& a, int n_pblocks, hipStream_t stream) {
  constexpr int PW = 64 * PPL;
  constexpr int kRed = STATS ? 3 : 2;
  const size_t lds = static_cast<size_t>(a.E) * PW * 4 + static_cast<size_t>(2) * TACG_MAX_REPLICATED * PW * 4 +
                     static_cast<size_t>(a.G) * PW * 2 + align256(a.E) +
                     static_cast<size_t>(kRed * PW + 1) * 4;
  allow_lds(&ev_main<K, PPL, STATS>, lds);
  EvArgs b = a;
  b.n_pblocks = n_pblocks;
  const int64_t grid = static_cast<int64_t>(n_pblocks) * a.n_pieces * a.L;
  if (grid > 0x7fffffff) return TACG_E_UNSUPPORTED;
  hipLaunchKernelGGL((ev_main<K, PPL, STATS>), dim3(static_cast<uint32_t>(grid)), dim3(kMainThreads), lds, stream,
                     b);
  return TACG_OK;
}

template <int K>
void launch_valid(const EvBase& a, const CountSegs& segs, hipStream_t stream) {
  // Eight workgroups per CU; fewer when a workgroup would see less than 2048 token-layers (its counts are flushed once).  A
  // short trace is bound by a workgroup's chain: segments (layers, with statistics their families), 2 to 5 us each, and steps.  So
  // at least two workgroups per segment, and one per step up to 256.  Whole statistics calls, one workgroup per 2048
  // token-layers against this: 64 families, 561 tokens x 4 layers, 64 placements 534 -> 49 us; 1939 tokens, 65 placements 353 -> 56 us;
  // 2^19 tokens x 4 layers of 8 experts are slower split further (46 against 54 us: more adds to few counters).
  const int64_t total = a.N * a.L, segments = static_cast<int64_t>(a.L) * (a.stats ? a.F : 1);
  const int64_t want = std::max({total / 2048, 2 * segments, std::min<int64_t>(total / 256, 256)});
  const int blocks = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(2048, want)));
  hipLaunchKernelGGL(ev_valid<K>, dim3(blocks), dim3(256), 0, stream, a, segs);
}

template <int K>
int launch_main_k(const EvArgs& a, hipStream_t stream) {
  // the statistics variant exists for two placements per lane only (it is not on the timed path)
  if (a.stats) return launch_main<K, 2, true>(a, (a.P + 127) / 128, stream);
  if (a.E > 64) return launch_main<K, 2, false>(a, (a.P + 127) / 128, stream);
  return launch_main<K, 4, false>(a, (a.P + 255) / 256, stream);
}

// Per-(placement, layer) primary-only loads from D.  A workgroup takes one layer and a run of placements: it sums
// the families' dispatches of every expert once, then each wave scores placements of its own, lanes over experts,
// into its own counters (64-bit LDS adds).  Bound by the latency of the table rows (four byte loads per
// placement, the next placement's in flight) and by LDS adds on few addresses.  Measured on MI355X at E = 256, 32
// GPUs, 16 families, 1024 placements x 58 layers: 140 -> 19 us (one workgroup per (placement, layer)
// summed the families again each time).
__global__ __launch_bounds__(64 * kLoadWaves) void placement_load_kernel(const uint32_t* __restrict__ D, int F, int L,
                                                                         int E, const uint8_t* __restrict__ primary,
                                                                         int P, int G, int run,
                                                                         int64_t* __restrict__ load_ref,
                                                                         uint32_t* d_err) {
  __shared__ unsigned long long acc[kLoadWaves][TACG_MAX_GPUS];
  __shared__ unsigned long long sum[TACG_MAX_EXPERTS];
  const int l = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int e = threadIdx.x; e < E; e += blockDim.x) {
    unsigned long long s = 0;
#pragma unroll 8
    for (int f = 0; f < F; ++f) s += D[(static_cast<int64_t>(f) * L + l) * E + e];
    sum[e] = s;
  }
  __syncthreads();
  unsigned long long d[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) d[q] = lane + 64 * q < E ? sum[lane + 64 * q] : 0ull;
  const int p1 = min(P, static_cast<int>(blockIdx.x + 1) * run);
  uint32_t err = 0;
  uint8_t next[4];
  auto fetch = [&](int p) {
    const uint8_t* src = primary + (static_cast<int64_t>(min(p, P - 1)) * L + l) * E;
#pragma unroll
    for (int q = 0; q < 4; ++q) next[q] = src[min(lane + 64 * q, E - 1)];
  };
  int p = blockIdx.x * run + wave;
  fetch(p);
  for (; p < p1; p += nw) {
    uint32_t g[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) g[q] = next[q];
    fetch(p + nw);
    if (lane < G) acc[wave][lane] = 0;
    __asm__ __volatile__("" ::: "memory");  // the LDS keeps a wave's operations in order
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (lane + 64 * q >= E) continue;
      if (g[q] >= static_cast<uint32_t>(G)) {
        err |= TACG_ERR_TABLE;
      } else if (d[q]) {
        __hip_atomic_fetch_add(&acc[wave][g[q]], d[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __asm__ __volatile__("" ::: "memory");
    if (lane < G) load_ref[(static_cast<int64_t>(p) * L + l) * G + lane] = static_cast<int64_t>(acc[wave][lane]);
  }
  if (err) atomicOr(d_err, err);
}

// Few placements: one workgroup per placement and layer, a thread per expert.  Up to kLoadFew of them nothing is worth sharing:
// placement_load, this / the kernel above at its best run, in us: 90 placements x 12 layers, E = 252, 2.8 / 3.3; 198 x 2, E =
// 128, 2.4 / 2.8; one GPU holding 252 experts, 35 x 1, 3.9 / 4.5; but 100 x 24, E = 256, 16 families, 5.9 / 4.6.
// grid (P, L), 256 threads.
constexpr int64_t kLoadFew = 1152;

__global__ __launch_bounds__(256) void placement_load_few_kernel(const uint32_t* __restrict__ D, int F, int L, int E,
                                                                 const uint8_t* __restrict__ primary, int G,
                                                                 int64_t* __restrict__ load_ref, uint32_t* d_err) {
  __shared__ unsigned long long acc[TACG_MAX_GPUS];
  const int p = blockIdx.x, l = blockIdx.y, tid = threadIdx.x;
  if (tid < G) acc[tid] = 0;
  __syncthreads();
  if (tid < E) {
    const uint32_t g = primary[(static_cast<int64_t>(p) * L + l) * E + tid];
    if (g < static_cast<uint32_t>(G)) {
      unsigned long long s = 0;
#pragma unroll 8
      for (int f = 0; f < F; ++f) s += D[(static_cast<int64_t>(f) * L + l) * E + tid];
      if (s) __hip_atomic_fetch_add(&acc[g], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
      atomicOr(d_err, TACG_ERR_TABLE);
    }
  }
  barrier_after_lds_atomics();
  if (tid < G) load_ref[(static_cast<int64_t>(p) * L + l) * G + tid] = static_cast<int64_t>(acc[tid]);
}

// Jain and MaxVio.  One wave per output row; lanes over GPUs.
__global__ __launch_bounds__(64) void jain_kernel(const uint32_t* __restrict__ load, int P, int L, int G,
                                                  int per_layer, float* __restrict__ jain, float* __restrict__ maxvio) {
  const int row = blockIdx.x;  // p (global) or p * L + l (per layer)
  const int m = threadIdx.x;
  uint64_t x = 0;
  if (per_layer) {
    if (m < G) x = load[static_cast<int64_t>(row) * G + m];
  } else {
    // the two halves of the wave take the even and the odd layers (G <= 32), several loads in flight
    const int c = min(m & 31, G - 1);
#pragma unroll 8
    for (int l = m >> 5; l < L; l += 2) x += load[(static_cast<int64_t>(row) * L + l) * G + c];
    x += __shfl_xor(x, 32, 64);
    if (m >= G) x = 0;
  }
  // exact integer sums; the square sum is formed in float64 (it can exceed 64 bits)
  uint64_t s = x, mx = x;
  double sq = static_cast<double>(x) * static_cast<double>(x);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    s += __shfl_xor(s, o, 64);
    const uint64_t other = __shfl_xor(mx, o, 64);
    mx = other > mx ? other : mx;
    sq += __shfl_xor(sq, o, 64);
  }
  if (m == 0) {
    const double tot = static_cast<double>(s);
    double j = 1.0, v = 0.0;
    if (s > 0) {
      j = tot * tot / (G * sq);
      const double mean = tot / G;
      v = (static_cast<double>(mx) - mean) / mean;
    }
    jain[row] = static_cast<float>(j);
    maxvio[row] = static_cast<float>(v);
  }
}

}  // namespace

// Placements per workgroup of the load passes: 64 share a layer's sums, but few placements are bound by a wave's chain of them,
// so they are spread until the chip holds about 512 workgroups.  placement_load at 8, 16, 32 and 64 per workgroup, device time in
// us: 90 placements x 12 layers, E = 252, 3.4, 4.2, 5.3 and 7.8 (3.3 at 4, one a wave); 400 x 12, E = 256, 16 families, 5.1, 5.4, 5.8 and 7.6; 256 x 58
// 8.9, 7.0, 7.0 and 7.8; 512 x 24, E = 60, 5.5, 4.3, 4.6 and 5.6; 1024 x 58 45.7, 28.5, 20.9 and 18.6.
struct LoadSplit {
  int waves, run;
};

static LoadSplit load_split(int32_t P, int32_t L) {
  const int64_t rows = static_cast<int64_t>(P) * L;
  if (rows <= 2048) return LoadSplit{4, 4};
  const int64_t run = rows / 512 / kLoadWaves * kLoadWaves;
  return LoadSplit{kLoadWaves, static_cast<int>(std::max<int64_t>(kLoadWaves, std::min<int64_t>(64, run)))};
}

size_t eval_workspace(int64_t n_tokens, int32_t L, int32_t E, int32_t G, int32_t P, int32_t F) {
  size_t used = 0;
  carve_ev(nullptr, n_tokens, L, E, G, P, F, &used);
  return used;
}

int launch_eval(const int16_t* trace, int64_t N, int32_t L, int32_t K, int32_t E, const int64_t* fam_off_host,
                int32_t F, const int32_t* home_start_host, const int32_t* home_size_host, int32_t G, int32_t P,
                const uint8_t* primary, const uint8_t* secondary, int32_t R, const int64_t* load_ref,
                int32_t theta_num, int32_t theta_den, uint64_t* cost_home, uint64_t* cost_span, uint32_t* load,
                uint64_t* cost_home_fam, const TraceStatsOut* stats, uint32_t* d_err, void* workspace,
                hipStream_t stream) {
  EvArgs a{};
  a.trace = trace;
  a.primary = primary;
  a.secondary = R > 0 ? secondary : nullptr;
  a.load_ref = load_ref;
  a.d_err = d_err;
  a.ws = carve_ev(workspace, N, L, E, G, P, F);
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
  a.stats = stats != nullptr;
  a.band_starts = stats != nullptr ? stats->band_starts : 0u;
  for (int f = 0; f < F; ++f) {
    const uint32_t bw = static_cast<uint32_t>(home_start_host[f]) | (static_cast<uint32_t>(home_size_host[f]) << 8);
    uint4& r = a.band4[f >> 2];
    ((f & 3) == 0 ? r.x : (f & 3) == 1 ? r.y : (f & 3) == 2 ? r.z : r.w) = bw;
  }
  // pieces: split every family's tokens into chunks sized for about kTargetWorkgroups workgroups of
  // ev_main (at least 4096 tokens; at most 2^26 so that the per-lane 32-bit cost accumulators cannot
  // overflow).
  const int64_t n_pblocks = (E > 64 || stats != nullptr) ? (P + 127) / 128 : (P + 255) / 256;
  int64_t chunk = (N * n_pblocks * L + kTargetWorkgroups - 1) / kTargetWorkgroups;
  chunk = std::min<int64_t>(int64_t(1) << 26, std::max<int64_t>(4096, chunk));
  int np = 0;
  for (;;) {
    np = 0;
    for (int f = 0; f < F; ++f) {
      const int64_t n = fam_off_host[f + 1] - fam_off_host[f];
      np += static_cast<int>((n + chunk - 1) / chunk);
    }
    if (np <= kMaxPieces || chunk >= (int64_t(1) << 26)) break;
    chunk = std::min<int64_t>(chunk * 2, int64_t(1) << 26);
  }
  if (np > kMaxPieces) return TACG_E_UNSUPPORTED;
  np = 0;
  for (int f = 0; f < F; ++f) {
    for (int64_t t = fam_off_host[f]; t < fam_off_host[f + 1]; t += chunk) {
      const int64_t e = std::min<int64_t>(t + chunk, fam_off_host[f + 1]);
      a.piece[np] = make_uint4(static_cast<uint32_t>(t), static_cast<uint32_t>(e),
                               static_cast<uint32_t>(fam_off_host[f]),
                               static_cast<uint32_t>(home_start_host[f]) |
                                   (static_cast<uint32_t>(home_size_host[f]) << 8) |
                                   (static_cast<uint32_t>(f) << 16));
      ++np;
    }
  }
  a.n_pieces = np;

  const EvBase& base = a;
  const dim3 block(256);
  if (static_cast<int64_t>(P) * E <= kPrepTables && (R == 0 || P <= kPrepPlace)) {
    switch (R) {
      case 0: hipLaunchKernelGGL(ev_prep<0>, dim3(L), block, 0, stream, base); break;
      case 1: hipLaunchKernelGGL(ev_prep<1>, dim3(L), block, 0, stream, base); break;
      case 2: hipLaunchKernelGGL(ev_prep<2>, dim3(L), block, 0, stream, base); break;
      case 3: hipLaunchKernelGGL(ev_prep<3>, dim3(L), block, 0, stream, base); break;
      default: hipLaunchKernelGGL(ev_prep<4>, dim3(L), block, 0, stream, base); break;
    }
  } else {
    hipLaunchKernelGGL(ev_zero, dim3(256), block, 0, stream, base);
    const int64_t n = static_cast<int64_t>(P) * L * E;
    const dim3 grid(static_cast<int>(std::min<int64_t>(2048, (n + 256 * kFlagsAhead - 1) / (256 * kFlagsAhead))));
    switch (R) {
      case 0: hipLaunchKernelGGL(ev_flags<0>, grid, block, 0, stream, base); break;
      case 1: hipLaunchKernelGGL(ev_flags<1>, grid, block, 0, stream, base); break;
      case 2: hipLaunchKernelGGL(ev_flags<2>, grid, block, 0, stream, base); break;
      case 3: hipLaunchKernelGGL(ev_flags<3>, grid, block, 0, stream, base); break;
      default: hipLaunchKernelGGL(ev_flags<4>, grid, block, 0, stream, base); break;
    }
    hipLaunchKernelGGL(ev_replist, dim3(L), block, 0, stream, base);
    if (R > 0) hipLaunchKernelGGL(ev_repinfo, dim3((P + 15) / 16, L), block, 0, stream, base);
  }
  if (hipGetLastError() != hipSuccess) return TACG_E_DEVICE;
  if (np > 0) {
    int32_t with_tokens = 0;
    for (int f = 0; f < F; ++f) with_tokens += fam_off_host[f + 1] > fam_off_host[f];
    const bool planes = stats == nullptr && eval_uses_planes(K, E, G, R, N, with_tokens);
    const bool tokens = eval_uses_tokens(P, R, planes, N, L, K, with_tokens);
    CountSegs segs;
    for (int f = 0; f < TACG_MAX_FAMILIES; ++f)
      segs.end[f] = f < F ? static_cast<uint32_t>(fam_off_host[f + 1]) : 0xffffffffu;
    int rc;
    switch (K) {
#define TACG_K(k) \
  case k:         \
    launch_valid<k>(a, segs, stream);  \
    rc = tokens   ? launch_eval_tokens(a, fam_off_host, home_start_host, home_size_host, stream) \
         : planes ? launch_eval_planes(a, fam_off_host, home_start_host, home_size_host, stream) \
                  : launch_main_k<k>(a, stream); \
    break;
      TACG_K(1) TACG_K(2) TACG_K(3) TACG_K(4) TACG_K(5) TACG_K(6) TACG_K(7) TACG_K(8)
      TACG_K(9) TACG_K(10) TACG_K(11) TACG_K(12) TACG_K(13) TACG_K(14) TACG_K(15) TACG_K(16)
#undef TACG_K
      default:
        return TACG_E_UNSUPPORTED;
    }
    if (rc != TACG_OK) return rc;
    if (hipGetLastError() != hipSuccess) return TACG_E_DEVICE;
  }
  const LoadSplit ls = load_split(P, L);
  hipLaunchKernelGGL(ev_finalize, dim3((P + ls.run - 1) / ls.run, L), dim3(64 * ls.waves), 0, stream, a, ls.run, cost_home,
                     cost_span, load, cost_home_fam);
  // four entries of (layer, expert) a thread: with idle waves a short table's launch takes longer (1024 placements x 16 families
  // of 2 x 160 entries: 57 us with 1024 threads)
  if (stats != nullptr)
    hipLaunchKernelGGL(ev_stats, dim3(P, F), dim3(std::min(1024, (L * E + 255) / 256 * 64)), 0, stream, a, stats->span_fam, stats->cross_fam,
                       stats->home_mass_fam);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

int launch_placement_load(const uint32_t* D, int32_t F, int32_t L, int32_t E, const uint8_t* primary, int32_t P,
                          int32_t G, int64_t* load_ref, uint32_t* d_err, hipStream_t stream) {
  if (static_cast<int64_t>(P) * L <= kLoadFew) {
    hipLaunchKernelGGL(placement_load_few_kernel, dim3(P, L), dim3(256), 0, stream, D, F, L, E, primary, G, load_ref, d_err);
    return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
  }
  const LoadSplit ls = load_split(P, L);
  hipLaunchKernelGGL(placement_load_kernel, dim3((P + ls.run - 1) / ls.run, L), dim3(64 * ls.waves), 0, stream, D, F, L, E,
                     primary, P, G, ls.run, load_ref, d_err);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

int launch_jain(const uint32_t* load, int32_t P, int32_t L, int32_t G, int32_t per_layer, float* jain,
                float* maxvio, hipStream_t stream) {
  const int rows = per_layer ? P * L : P;
  hipLaunchKernelGGL(jain_kernel, dim3(rows), dim3(64), 0, stream, load, P, L, G, per_layer, jain, maxvio);
  return hipGetLastError() == hipSuccess ? TACG_OK : TACG_E_DEVICE;
}

}  // namespace tacg
