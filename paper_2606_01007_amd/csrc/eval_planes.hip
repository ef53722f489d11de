// Placement scoring on bit planes: the trace pass of tacg_eval_placements for at most 8 GPUs.
//
// A dword holds one bit of each of 32 placements (a "group"), and the one-hot GPU of an expert is NP such
// planes (NP = 4 or 8 >= G), so a token-layer's GPU set over 32 placements is the OR of its experts' planes:
// per lane and 8-expert token 32 three-input ORs and 256 bytes of LDS reads, where the lane = placement pass
// (eval.hip) spends 32 x 4 ORs, 1 KB of LDS reads and 32 x 3 counting operations.
//
// Work split: the tokens of a family that share one anchor GPU (t = pos mod band size) form a class, cut into
// tiles of 64 tokens; a workgroup scores up to 16 groups (512 placements) of one layer on an equal share of
// the layer's tiles.  It walks the classes that its share crosses, so the anchor is fixed within a run, and
// the tables are built once.
// Lanes hold (token slot, group): with 2^b groups, 64 / 2^b tokens per wave step, and lane c of every row
// of 16 lanes always reads column c of the LDS tables (column c holds group c mod 2^b).
//
// LDS tables, 256-byte rows of 16 columns x 4 planes (one 16-byte read serves a lane; the 16 lanes of a
// row of lanes read one 256-byte row, so every read is free of bank conflicts whatever the experts are):
//   tbl[e][NP/4]    one-hot GPU planes of expert e where it has a single candidate, else 0; row E is zero
//   rep[r][2 NP/4]  feasible-candidate planes of replicated expert r, then the one-hot planes of its choice when no
//                   feasible candidate is reached (the anchor if feasible, else the least-loaded); row 16 is zero
//
// A wave prepares 64 tokens at once (one per lane): ids to 16-bit table rows, the replicated slots' rows in
// slot order, and a stable sort by the number of replicated slots (invalid tokens last, on the zero rows),
// so that a step's tokens have nearly equal numbers of them.  A step then ORs the planes, resolves the
// replicated slots in slot order (lowest reached feasible GPU by a priority chain over the planes), and adds
// the planes to vertical counters: bit-sliced carry-save sums whose level i is touched every 2^i steps.  The GPU counts of the
// replicated choices are first transposed across the wave's four rows of lanes, so that each row counts its
// own NP / 4 GPUs.  At the end the vertical counters are transposed to one integer per placement.
//
// What bounds it: VALU issue and LDS reads about equally (top-8, one replicated slot per token: about 185 VALU
// instructions and 25 16-byte reads per step of 64 lanes; three waves per SIMD hide most of the latency).
// Measured on MI355X against the lane = placement pass, whole tacg_eval_placements calls: E = 128, top-8, 8 GPUs,
// 1024 placements with 8 x 2 replicas, 2^18 tokens x 48 layers: 9.56 -> 2.51 ms; E = 60, top-4, 6 GPUs, 512
// placements with 4 x 2, 120007 tokens x 24 layers: 0.711 -> 0.311 ms.
#include "eval_internal.h"

namespace tacg {
namespace {

constexpr int kThreads = 768;          // three waves per SIMD (up to 168 registers); 512 where the LDS is short
constexpr int kThreadsSmall = 512;
constexpr int kCols = 16;              // columns of a table row (one per lane of a row of lanes)
constexpr int kRowB = 256;             // bytes of a table row of four planes
constexpr int kRepRows = TACG_MAX_REPLICATED + 1;
constexpr int64_t kMaxTiles = 960;     // tiles per workgroup: at most 1920 steps per wave
constexpr size_t kLdsMax = 163840;

struct FamRec {  // 16-byte records (runtime-indexed kernel arguments)
  uint32_t off, end, first_tile, band;  // band: home_start | home_size << 8
};

struct PlArgs {
  const int16_t* trace;
  const uint8_t* primary;
  EvWs ws;
  int64_t N;
  int32_t L, E, F, G, P;
  int32_t n_shares, n_pblocks, n_full;  // n_full blocks of 16 groups, then the blocks of `tail`
  uint32_t n_tiles;                     // tiles of a layer (a class's last one may be short or empty)
  uint32_t tail[4];                     // first group | number of groups << 24
  FamRec fam[TACG_MAX_FAMILIES + 1];
};
static_assert(sizeof(PlArgs) <= 4096, "kernel arguments must stay within 4 KB");

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// Full adder over 32 placements: sum replaces a, returns the carry.
__device__ __forceinline__ uint32_t full_add(uint32_t& a, uint32_t b, uint32_t c) {
  const uint32_t carry = maj3(a, b, c);
  a = xor3(a, b, c);
  return carry;
}

// Vertical counter of planes.  Push number n (wave-uniform) adds one plane: level i < kLo is a running plane
// and a pending one, combined every 2^(i+1) pushes; every 2^kLo pushes the carry ripples through HI planes.
// Holds 2^(kLo + HI) - 1 pushes.
constexpr int kLo = 4;
constexpr int kSteps = 11;  // log2 of a bound of a wave's steps: see kMaxTiles

template <int HI>
struct VCount {
  uint32_t run[kLo + HI], pend[kLo];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < kLo + HI; ++i) run[i] = 0;
#pragma unroll
    for (int i = 0; i < kLo; ++i) pend[i] = 0;
  }
};

// Push number n of M counters at once (they share the branches on n).
template <int M, int HI, int I = 0>
__device__ __forceinline__ void push(VCount<HI> (&c)[M], const uint32_t (&x)[M], uint32_t n) {
  if constexpr (I < kLo) {
    if ((n >> I) & 1u) {
      uint32_t y[M];
#pragma unroll
      for (int k = 0; k < M; ++k) y[k] = full_add(c[k].run[I], c[k].pend[I], x[k]);
      push<M, HI, I + 1>(c, y, n);
    } else {
#pragma unroll
      for (int k = 0; k < M; ++k) c[k].pend[I] = x[k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < M; ++k) {
      uint32_t y = x[k];
#pragma unroll
      for (int i = kLo; i < kLo + HI; ++i) {
        const uint32_t t = c[k].run[i] & y;
        c[k].run[i] ^= y;
        y = t;
      }
    }
  }
}

template <int S>
__device__ __forceinline__ void swap_bits(uint32_t (&v)[32]) {
  constexpr uint32_t m = S == 4 ? 0x0f0f0f0fu : S == 2 ? 0x33333333u : 0x55555555u;
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    if (k & S) continue;
    const uint32_t lo = v[k], hi = v[k + S];
    v[k] = (lo & m) | ((hi << S) & ~m);
    v[k + S] = ((lo >> S) & m) | (hi & ~m);
  }
}

// 32 x 32 bit transpose: bit j of v[i] becomes bit i of v[j].
__device__ __forceinline__ void transpose32(uint32_t (&v)[32]) {
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const uint32_t lo = v[k], hi = v[k + 16];
    v[k] = __builtin_amdgcn_perm(hi, lo, 0x05040100);
    v[k + 16] = __builtin_amdgcn_perm(hi, lo, 0x07060302);
  }
#pragma unroll
  for (int b = 0; b < 32; b += 16) {
#pragma unroll
    for (int k = b; k < b + 8; ++k) {
      const uint32_t lo = v[k], hi = v[k + 8];
      v[k] = __builtin_amdgcn_perm(hi, lo, 0x06020400);
      v[k + 8] = __builtin_amdgcn_perm(hi, lo, 0x07030501);
    }
  }
  swap_bits<4>(v);
  swap_bits<2>(v);
  swap_bits<1>(v);
}

// Values of a vertical counter after n pushes of weight 2^LOW, with LOW lower planes: out[j] for placement j.
template <int LOW, int HI>
__device__ __forceinline__ void read_counter(const uint32_t* low, const VCount<HI>& c, uint32_t n, uint32_t (&v)[32]) {
  static_assert(LOW + kLo + HI <= 20 && LOW + kLo <= 12, "the counter and its pending planes share a dword");
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = 0;
#pragma unroll
  for (int i = 0; i < LOW; ++i) v[i] = low[i];
#pragma unroll
  for (int i = 0; i < kLo + HI; ++i) v[LOW + i] = c.run[i];
#pragma unroll
  for (int i = 0; i < kLo; ++i) v[20 + LOW + i] = ((n >> i) & 1u) ? c.pend[i] : 0u;
  transpose32(v);
#pragma unroll
  for (int j = 0; j < 32; ++j) v[j] = (v[j] & 0xfffffu) + (v[j] >> 20);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// LDS reads by byte offset.  The kernel's only LDS is its dynamic array, which starts at LDS address 0; with
// plain integer addresses the constant part of an offset goes into the instruction.
__device__ __forceinline__ u32x4 lds_read16(uint32_t off) {
  return *(__attribute__((address_space(3))) const u32x4*)(uintptr_t)off;
}
__device__ __forceinline__ u32x2 lds_read8(uint32_t off) {
  return *(__attribute__((address_space(3))) const u32x2*)(uintptr_t)off;
}

template <int NP>
__device__ __forceinline__ void load_planes(uint32_t off, uint32_t (&v)[NP]) {
#pragma unroll
  for (int q = 0; q < NP / 4; ++q) {
    const u32x4 x = lds_read16(off + q * kRowB);
    v[4 * q] = x.x;
    v[4 * q + 1] = x.y;
    v[4 * q + 2] = x.z;
    v[4 * q + 3] = x.w;
  }
}

template <int K, int NP>
struct PlLayout {
  static constexpr int NQ = NP / 4;                    // 256-byte rows per expert
  static constexpr int RS = 2 * NQ;                    // rows per replicated expert
  static constexpr int KW = (K + 1) / 2;               // dwords of 16-bit table rows per token
  static constexpr int KR = (K + 3) / 4;               // dwords of 8-bit replica rows per token
  static constexpr int DW = (KW + KR + 1) / 2 * 2;     // dwords of a token's descriptor (8-byte multiple)
  static constexpr uint32_t kNull = TACG_MAX_REPLICATED * RS;  // replica row of an unused slot (zero)
  static constexpr int kRepBytes = kRepRows * RS * kRowB;
  static constexpr int kRed = NP * kCols * 32;         // dwords of the final sums of the choices
  static int desc_off(int E) { return kRepBytes + (E + 1) * NQ * kRowB; }
  static size_t bytes(int E, int threads) {
    size_t b = static_cast<size_t>(desc_off(E)) + static_cast<size_t>(threads) * DW * 4;
    b = std::max(b, static_cast<size_t>(kRed) * 4);
    return b + 256;  // rep_of
  }
  static int threads(int E) { return bytes(E, kThreads) <= kLdsMax ? kThreads : kThreadsSmall; }
};

// grid (layers x shares x placement blocks, placement block fastest), PlLayout::threads
template <int K, int NP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void ev_planes(PlArgs a) {
  using Lay = PlLayout<K, NP>;
  constexpr int NQ = Lay::NQ, RS = Lay::RS, KW = Lay::KW, KR = Lay::KR, DW = Lay::DW;
  constexpr int NJ = NP / 4;  // GPUs counted per row of lanes
  extern __shared__ __align__(16) char lds[];
  const int E = a.E, G = a.G, L = a.L, P = a.P;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthreads = blockDim.x, nwaves = nthreads >> 6;
  // XCD-aware order, as in ev_main: the placement blocks of one (piece, layer) run together on one XCD
  const uint32_t total = gridDim.x, b = blockIdx.x;
  const uint32_t xcd = b % kXcds, per = total / kXcds, rem = total % kXcds;
  const uint32_t vid = xcd * per + min(xcd, rem) + b / kXcds;
  const int pb = static_cast<int>(vid % a.n_pblocks);
  const uint32_t ls = vid / a.n_pblocks;
  const uint32_t share = ls % a.n_shares;
  const int l = ls / a.n_shares;
  uint32_t x0 = static_cast<uint32_t>(static_cast<uint64_t>(a.n_tiles) * share / a.n_shares);
  const uint32_t x1 = static_cast<uint32_t>(static_cast<uint64_t>(a.n_tiles) * (share + 1) / a.n_shares);
  if (x0 == x1) return;
  const uint32_t share0 = x0;
  int g0 = pb * kCols, ngrp = kCols;
  if (pb >= a.n_full) {
    const uint32_t t = a.tail[pb - a.n_full];
    g0 = t & 0xffffff;
    ngrp = t >> 24;
  }
  char* const rep = lds;
  char* const tbl = lds + Lay::kRepBytes;
  const size_t tbl_end = Lay::kRepBytes + static_cast<size_t>(E + 1) * NQ * kRowB;
  uint32_t* const desc = reinterpret_cast<uint32_t*>(lds + tbl_end);
  size_t tail_off = tbl_end + static_cast<size_t>(nthreads) * DW * 4;
  if (tail_off < static_cast<size_t>(Lay::kRed) * 4) tail_off = static_cast<size_t>(Lay::kRed) * 4;
  uint8_t* const rep_of = reinterpret_cast<uint8_t*>(lds + tail_off);
  const uint8_t* rep_of_g = a.ws.rep_of + static_cast<int64_t>(l) * E;
  const int nrep = a.ws.n_rep[l];

  // ---- tables ----
  for (int e = tid; e < E; e += nthreads) rep_of[e] = rep_of_g[e];
  for (int i = tid; i < NQ * kRowB / 4; i += nthreads) reinterpret_cast<uint32_t*>(tbl + E * NQ * kRowB)[i] = 0;
  for (int i = tid; i < RS * kRowB / 4; i += nthreads)
    reinterpret_cast<uint32_t*>(rep + Lay::kNull * kRowB)[i] = 0;
  {
    // one-hot planes: a wave takes 64 experts of one group (the 64 lanes read consecutive bytes)
    const int nch = (E + 63) / 64;
    for (int it = wave; it < ngrp * nch; it += nwaves) {
      const int c = it / nch, e = (it - c * nch) * 64 + lane;
      if (e >= E) continue;
      const int p0 = min((g0 + c) * 32, P - 1);  // a padded group of the last block has no placement
      const int np = min(32, P - (g0 + c) * 32), last = max(np, 1) - 1;
      const uint8_t* src = a.primary + (static_cast<int64_t>(p0) * L + l) * E + e;
      const int64_t stride = static_cast<int64_t>(L) * E;
      uint32_t b0 = 0, b1 = 0, b2 = 0;
#pragma unroll
      for (int q0 = 0; q0 < 32; q0 += 16) {
        uint32_t x[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = src[min(q0 + q, last) * stride];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          b0 |= (x[q] & 1u) << (q0 + q);
          b1 |= ((x[q] >> 1) & 1u) << (q0 + q);
          if constexpr (NP > 4) b2 |= ((x[q] >> 2) & 1u) << (q0 + q);
        }
      }
      uint32_t on = np >= 32 ? ~0u : np > 0 ? (1u << np) - 1u : 0u;
      const uint32_t r = rep_of_g[e];
      if (r != kNone) {  // zero where the expert has several candidates
        const uint2* ri = a.ws.rep_info + (static_cast<int64_t>(l) * TACG_MAX_REPLICATED + r) * P + p0;
        uint32_t single = 0;
#pragma unroll
        for (int q0 = 0; q0 < 32; q0 += 16) {
          uint32_t y[16];
#pragma unroll
          for (int q = 0; q < 16; ++q) y[q] = ri[min(q0 + q, last)].y;
#pragma unroll
          for (int q = 0; q < 16; ++q) single |= (y[q] >> 31) << (q0 + q);
        }
        on &= single;
      }
      uint32_t pl[NP];
      const uint32_t lo[4] = {on & ~b0 & ~b1, on & b0 & ~b1, on & ~b0 & b1, on & b0 & b1};
#pragma unroll
      for (int g = 0; g < NP; ++g) pl[g] = NP == 4 ? lo[g] : lo[g & 3] & ((g & 4) ? b2 : ~b2);
      for (int cc = c; cc < kCols; cc += ngrp) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          *reinterpret_cast<uint4*>(tbl + (e * NQ + q) * kRowB + cc * 16) =
              make_uint4(pl[4 * q], pl[4 * q + 1], pl[4 * q + 2], pl[4 * q + 3]);
      }
    }
  }
  // replica rows: a wave takes 64 placements (two groups) of one replicated expert, one per lane; the candidate
  // planes (part 0) once, the planes of the choice when none is reached (part 1) for every anchor
  auto rep_rows = [&](int part, uint32_t h) {
    const int npair = (ngrp + 1) / 2;
    for (int it = wave; it < nrep * npair; it += nwaves) {
      const int r = it / npair, c = 2 * (it - r * npair);
      const int p = (g0 + c) * 32 + lane;
      const bool live = p < P;
      const uint2 v = live ? a.ws.rep_info[(static_cast<int64_t>(l) * TACG_MAX_REPLICATED + r) * P + p] : make_uint2(0u, 0u);
      const uint32_t alt = ((v.x >> h) & 1u) ? h : (v.y & 31u);
      const uint32_t bits = part == 0 ? v.x : live ? 1u << alt : 0u;
      const int cl = lane & (ngrp - 1);  // lanes 0..15 write the copies of the two columns
      const bool wr = lane < kCols && (cl >> 1) == (c >> 1);
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        const uint64_t bal = __ballot(((bits >> m) & 1u) != 0u);
        const uint32_t w = (cl & 1) ? static_cast<uint32_t>(bal >> 32) : static_cast<uint32_t>(bal);
        if (wr)
          *reinterpret_cast<uint32_t*>(rep + (r * RS + part * NQ + (m >> 2)) * kRowB + lane * 16 + (m & 3) * 4) = w;
      }
    }
  };
  rep_rows(0, 0u);

  const bool any_bad = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(*a.ws.n_bad != 0u)) != 0u;
  const int lg = __builtin_ctz(ngrp);             // log2 groups
  const int slots = 64 >> lg;                     // tokens per step
  const uint32_t slot = static_cast<uint32_t>(lane) >> lg;
  const uint32_t col = static_cast<uint32_t>(lane & 15) * 16u;
  uint32_t* const wdesc = desc + wave * 64 * DW;
  const uint32_t wdesc_off = static_cast<uint32_t>(tbl_end) + wave * 64 * DW * 4;

  VCount<kSteps - kLo + (K > 8 ? 4 : 3)> pick[NJ];  // a step has at most K replicated slots
  uint32_t plow[NJ][2];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    pick[j].clear();
    plow[j][0] = plow[j][1] = 0;
  }
  uint32_t n_pick = 0;  // pushes so far (wave-uniform)
  const int row16 = lane >> 4;
  // GPU counted by this lane's row as its j-th (see the swaps below)
  auto pick_gpu = [&](int j) { return NP == 4 ? ((row16 >> 1) * 2 + (row16 & 1)) : (row16 >> 1) * 4 + (row16 & 1) * 2 + j; };

  auto add_all = [&](uint32_t* dst, const uint32_t (&v)[32]) {
#pragma unroll
    for (int q = 0; q < 32; ++q)
      __hip_atomic_fetch_add(dst + q * kCols + (lane & 15), v[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  int f = 0;
  while (x0 < x1) {
    // ---- the run of this share's tiles in one class ----
    while (a.fam[f + 1].first_tile <= x0) ++f;
    const FamRec fr = a.fam[f];
    const uint32_t hs = fr.band & 0xffu, hz = fr.band >> 8;
    const uint32_t n_f = fr.end - fr.off;
    const uint32_t per_class = (n_f - 1) / hz / 64 + 1;          // tiles of a class (the run has a tile: n_f > 0)
    const uint32_t pos = (x0 - fr.first_tile) / per_class;
    const uint32_t class0 = fr.first_tile + pos * per_class;
    const uint32_t xe = min(x1, class0 + per_class);
    const uint32_t h = hs + pos;
    const uint32_t c0 = (x0 - class0) * 64;                      // first token of the run, within the class
    uint32_t c1 = n_f > pos ? (n_f - pos - 1) / hz + 1 : 0u;     // the class's tokens
    if (xe - class0 < per_class) c1 = min(c1, (xe - class0) * 64);
    // the waves take the share's tiles in turn, across runs (so none exceeds its part of kMaxTiles)
    const uint32_t first = (wave + nwaves - (x0 - share0) % nwaves) % nwaves;
    x0 = xe;
    if (c0 >= c1) continue;
    rep_rows(1, h);
    uint32_t hm[NP];  // all ones for the anchor's plane
#pragma unroll
    for (int g = 0; g < NP; ++g) hm[g] = static_cast<uint32_t>(__builtin_amdgcn_sbfe(1 << h, g, 1));
    uint32_t low[NP == 4 ? 2 : 3];       // span: planes of weight 1, 2 (and 4)
    VCount<kSteps - kLo> cost[2];        // span above `low`, hits of the anchor
#pragma unroll
    for (int i = 0; i < (NP == 4 ? 2 : 3); ++i) low[i] = 0;
    cost[0].clear();
    cost[1].clear();
    uint32_t n_step = 0;  // pushes so far (wave-uniform)
    const int16_t* trace_c = a.trace + (static_cast<int64_t>(l) * a.N + fr.off + pos + static_cast<int64_t>(c0) * hz) * K;
    const uint32_t n_run = c1 - c0, ntile = (n_run + 63) / 64;   // at most kMaxTiles tiles
    TraceIds<K> next;  // the ids of the wave's next tile, in flight while the current one is scored
    next.fetch(trace_c + static_cast<int64_t>(min(first * 64 + lane, n_run - 1)) * hz * K);
    __syncthreads();  // the tables are in place
    for (uint32_t tile = first; tile < ntile; tile += nwaves) {
    // ---- one token per lane: descriptor, sorted by the number of replicated slots ----
    const uint32_t ci = tile * 64 + lane;  // within the run: a class may end just below 2^32
    const bool in = ci < n_run;
    uint32_t nvalid;
    {
      uint32_t raw[K];
      next.unpack(raw);
      next.fetch(trace_c + static_cast<int64_t>(min(ci + nwaves * 64, n_run - 1)) * hz * K);
      bool ok = in;
      if (any_bad) {  // some token-layer of the trace is invalid: leave those out
        bool dup = false;
#pragma unroll
        for (int s = 0; s < K; ++s) {
          ok &= raw[s] < static_cast<uint32_t>(E);
#pragma unroll
          for (int q = 0; q < s; ++q) dup |= raw[s] == raw[q];
        }
        ok &= !dup;
      }
      uint32_t d[DW];
#pragma unroll
      for (int i = 0; i < DW; ++i) d[i] = 0;
#pragma unroll
      for (int i = 0; i < KR; ++i) d[KW + i] = Lay::kNull * 0x01010101u;
      uint32_t cnt = 0;
#pragma unroll
      for (int s = 0; s < K; ++s) {
        const uint32_t id = ok ? raw[s] : static_cast<uint32_t>(E);
        d[s >> 1] |= (id * NQ) << (16 * (s & 1));
        const uint32_t r = ok && nrep > 0 ? rep_of[id] : kNone;
        if (r != kNone) {
          const uint32_t x = ((r * RS) ^ Lay::kNull) << (8 * (cnt & 3));
#pragma unroll
          for (int i = 0; i < KR; ++i) d[KW + i] ^= (static_cast<int>(cnt >> 2) == i) ? x : 0u;
          ++cnt;
        }
      }
      uint32_t place = 0, base = 0;
      uint64_t left = __ballot(ok);
      nvalid = __popcll(left);
      for (uint32_t c = 0; left != 0; ++c) {  // at most K + 1 passes: every valid token has cnt <= K
        const uint64_t m = __ballot(ok && cnt == c);
        if (ok && cnt == c) place = base + __popcll(m & ((1ull << lane) - 1ull));
        base += __popcll(m);
        left &= ~m;
      }
      const uint64_t bad = __ballot(!ok);
      if (!ok) place = nvalid + __popcll(bad & ((1ull << lane) - 1ull));
#pragma unroll
      for (int i = 0; i < DW / 2; ++i)
        *reinterpret_cast<uint2*>(wdesc + place * DW + 2 * i) = make_uint2(d[2 * i], d[2 * i + 1]);
    }
    // the steps below read what other lanes of this wave stored: the LDS executes a wave's operations in
    // order, so only the compiler has to keep them in order
    __builtin_amdgcn_wave_barrier();
    __asm__ __volatile__("" ::: "memory");

    uint32_t doff = wdesc_off + slot * (DW * 4);  // this lane's descriptor of the next step
    for (uint32_t j0 = 0; j0 < nvalid; j0 += slots, doff += slots * (DW * 4)) {
      uint32_t d[DW];
#pragma unroll
      for (int i = 0; i < DW / 2; ++i) {
        const u32x2 v = lds_read8(doff + 8 * i);
        d[2 * i] = v.x;
        d[2 * i + 1] = v.y;
      }
      // the planes of four slots in flight: the reads of slots s + 2, s + 3 go out before slots s, s + 1 are
      // OR-ed (byte offset of a row = its 16-bit number << 8 | column)
      uint32_t m[NP], v[4][NP];
#pragma unroll
      for (int g = 0; g < NP; ++g) m[g] = 0;
#pragma unroll
      for (int s = 0; s < K + 2; s += 2) {
#pragma unroll
        for (int u = s; u < s + 2; ++u)
          if (u < K)
            load_planes<NP>(Lay::kRepBytes + __builtin_amdgcn_perm(d[u >> 1], col, (u & 1) ? 0x0c070600u : 0x0c050400u), v[u & 3]);
        __builtin_amdgcn_sched_barrier(0);
        if (s >= 2) {
#pragma unroll
          for (int g = 0; g < NP; ++g) m[g] |= v[(s - 2) & 3][g] | (s - 1 < K ? v[(s - 1) & 3][g] : 0u);
        }
      }
      // replicated slots in slot order
#pragma unroll 1
      for (int i = 0; i < K; ++i) {
        const uint32_t r = d[KW] & 0xffu;
        if (__ballot(r != Lay::kNull) == 0) break;
        const uint32_t rp = __builtin_amdgcn_perm(d[KW], col, 0x0c0c0400u);
#pragma unroll
        for (int q = 0; q + 1 < KR; ++q) d[KW + q] = __builtin_amdgcn_alignbit(d[KW + q + 1], d[KW + q], 8);
        d[KW + KR - 1] = (d[KW + KR - 1] >> 8) | (Lay::kNull << 24);
        uint32_t fc[NP], alt[NP], pk[NP];
        load_planes<NP>(rp, fc);
        load_planes<NP>(rp + NQ * kRowB, alt);
        uint32_t seen = 0;
#pragma unroll
        for (int g = 0; g < NP; ++g) {
          pk[g] = __builtin_amdgcn_bitop3_b32(fc[g], m[g], seen, 0x40);  // fc & m & ~seen
          seen = __builtin_amdgcn_bitop3_b32(seen, fc[g], m[g], 0xF8);   // seen | (fc & m)
        }
#pragma unroll
        for (int g = 0; g < NP; ++g) {
          pk[g] = __builtin_amdgcn_bitop3_b32(pk[g], alt[g], seen, 0xF4);  // pk | (alt & ~seen)
          m[g] |= pk[g];
        }
        // transpose across the four rows of lanes: row w keeps its NP / 4 GPUs of all four rows
#pragma unroll
        for (int g = 0; g < NP / 2; ++g) {
          const auto s = __builtin_amdgcn_permlane32_swap(pk[g], pk[g + NP / 2], false, false);
          pk[g] = s[0];
          pk[g + NP / 2] = s[1];
        }
#pragma unroll
        for (int hh = 0; hh < NP; hh += NP / 2) {
#pragma unroll
          for (int g = 0; g < NP / 4; ++g) {
            const auto s = __builtin_amdgcn_permlane16_swap(pk[hh + g], pk[hh + g + NP / 4], false, false);
            pk[hh + g] = s[0];
            pk[hh + g + NP / 4] = s[1];
          }
        }
        uint32_t up[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const uint32_t ca = full_add(plow[j][0], pk[j], pk[j + NJ]);
          const uint32_t cb = full_add(plow[j][0], pk[j + 2 * NJ], pk[j + 3 * NJ]);
          up[j] = full_add(plow[j][1], ca, cb);
        }
        push(pick, up, n_pick);
        ++n_pick;
      }
      // costs: |cards| into the span counter, the anchor's plane into the hit counter
      uint32_t hit = 0;
#pragma unroll
      for (int g = 0; g < NP; ++g) hit |= m[g] & hm[g];
      uint32_t up[2] = {0u, hit};
      if constexpr (NP == 4) {
        const uint32_t ca = full_add(low[0], m[0], m[1]);
        const uint32_t cb = full_add(low[0], m[2], m[3]);
        up[0] = full_add(low[1], ca, cb);
      } else {
        const uint32_t ca = full_add(low[0], m[0], m[1]);
        const uint32_t cb = full_add(low[0], m[2], m[3]);
        const uint32_t cc = full_add(low[0], m[4], m[5]);
        const uint32_t cd = full_add(low[0], m[6], m[7]);
        const uint32_t da = full_add(low[1], ca, cb);
        const uint32_t db = full_add(low[1], cc, cd);
        up[0] = full_add(low[2], da, db);
      }
      push(cost, up, n_step);
      ++n_step;
    }
    __builtin_amdgcn_wave_barrier();
    __asm__ __volatile__("" ::: "memory");
  }

    // ---- the run's costs: per-placement sums of the workgroup in LDS (over the descriptors), one add each ----
    __syncthreads();
    for (int i = tid; i < 2 * 32 * kCols; i += nthreads) desc[i] = 0;
    __syncthreads();
    if (n_step > 0) {
      uint32_t v[32];
      read_counter<(NP == 4 ? 2 : 3)>(low, cost[0], n_step, v);
      add_all(desc, v);
      read_counter<0>(nullptr, cost[1], n_step, v);
      add_all(desc + 32 * kCols, v);
    }
    barrier_after_lds_atomics();
    for (int i = tid; i < ngrp * 32; i += nthreads) {
      // placement q of group c: the sum over the columns that hold group c
      const int c = i & (ngrp - 1), q = i >> lg, p = (g0 + c) * 32 + q;
      if (p >= P) continue;
      uint32_t sp = 0, hit = 0;
      for (int cc = c; cc < kCols; cc += ngrp) {
        sp += desc[q * kCols + cc];
        hit += desc[(32 + q) * kCols + cc];
      }
      const uint32_t away = sp - hit;
      if (sp) atomicAdd(&a.ws.acc_span[p], static_cast<unsigned long long>(sp));
      if (away) {
        atomicAdd(&a.ws.acc_home[p], static_cast<unsigned long long>(away));
        atomicAdd(&a.ws.acc_fam[static_cast<int64_t>(f) * P + p], static_cast<unsigned long long>(away));
      }
    }
    __syncthreads();
  }

  // ---- the choices of the replicated experts, summed over the tables ----
  if (nrep > 0) {
    uint32_t* const red = reinterpret_cast<uint32_t*>(lds);  // [NP][32][16]
    __syncthreads();
    for (int i = tid; i < Lay::kRed; i += nthreads) red[i] = 0;
    __syncthreads();
    if (n_pick > 0) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        uint32_t v[32];
        read_counter<2>(plow[j], pick[j], n_pick, v);
        add_all(red + pick_gpu(j) * 32 * kCols, v);
      }
    }
    barrier_after_lds_atomics();
    for (int i = tid; i < G * ngrp * 32; i += nthreads) {
      const int c = i & (ngrp - 1), gq = i >> lg, p = (g0 + c) * 32 + (gq & 31);
      if (p >= P) continue;
      uint32_t s = 0;
      for (int cc = c; cc < kCols; cc += ngrp) s += red[gq * kCols + cc];
      if (s) atomicAdd(a.ws.rep_load + (static_cast<int64_t>(l) * G + (gq >> 5)) * even_up(P) + p, s);
    }
  }
}

template <int K, int NP>
int launch_t(const PlArgs& a, hipStream_t stream) {
  const int threads = PlLayout<K, NP>::threads(a.E);
  const size_t lds = PlLayout<K, NP>::bytes(a.E, threads);
  if (lds > kLdsMax) return TACG_E_UNSUPPORTED;
  allow_lds(&ev_planes<K, NP>, lds);
  const int64_t grid = static_cast<int64_t>(a.n_pblocks) * a.n_shares * a.L;
  if (grid > 0x7fffffff) return TACG_E_UNSUPPORTED;
  hipLaunchKernelGGL((ev_planes<K, NP>), dim3(static_cast<uint32_t>(grid)), dim3(threads), lds, stream, a);
  return TACG_OK;
}

// Shares of a layer's tiles: workgroups of about equal work that fill whole rounds of the 256 CUs (one
// workgroup per CU).  A workgroup's set-up and flushes cost about as much as kSetup tiles of 16 groups (an estimate from the
// times of short and long inputs, not swept), so few rounds are best for short inputs; from 8 rounds on the last one no longer matters.
int64_t shares_of(int64_t tiles, int64_t rows, int groups) {
  constexpr int64_t kCus = 256, kSetup = 24;
  const int64_t floor_shares = (tiles + kMaxTiles - 1) / kMaxTiles;
  int64_t best = floor_shares, best_cost = INT64_MAX;
  for (int rounds = 1; rounds <= 8; ++rounds) {
    const int64_t s = std::min(tiles, std::max(floor_shares, rounds * kCus / rows));
    if (s < 1) continue;
    const int64_t used = (rows * s + kCus - 1) / kCus;                           // rounds of workgroups
    const int64_t cost = used * ((tiles + s - 1) / s * (groups + 2) + kSetup * (kCols + 2));
    if (cost < best_cost) {
      best_cost = cost;
      best = s;
    }
  }
  return std::max<int64_t>(best, 1);
}

template <int K>
size_t lds_k(int E, int G) {
  return G <= 4 ? PlLayout<K, 4>::bytes(E, kThreadsSmall) : PlLayout<K, 8>::bytes(E, kThreadsSmall);
}

}  // namespace

// At most 8 GPUs (a plane per GPU: the LDS reads and the planes of a token grow with their number; 8 took a third of the
// lane = placement pass's time, see above), and the tables of all experts within the 160 KB of LDS: every size with at most 4
// GPUs or top-8; with 5 to 8 GPUs up to 252 experts at top-9 and top-10, 244 at top-11 and top-12, and 236 above.
// Not for few experts without replicas, a short choice and short families, where the other pass's tables and steps are small and a
// class's set-up and flush are most of this one: E = 16, top-2, 512 placements, 24 layers, this pass against the other, 64 families
// of 8 tokens 104 / 77 us, 16 of 128 58 / 48 us, 64 of 128 129 / 136 us; 2 layers, 64 families of 64 tokens 32 / 23 us (E =
// 60, top-4: 32 / 32 us).
bool eval_uses_planes(int32_t K, int32_t E, int32_t G, int32_t n_sec, int64_t n_tokens, int32_t families_with_tokens) {
  if (G > 8) return false;
  if (E <= 32 && K <= 2 && n_sec == 0 && n_tokens <= int64_t(128) * families_with_tokens) return false;
  switch (K) {
#define TACG_K(k) \
  case k:         \
    return lds_k<k>(E, G) <= kLdsMax;
    TACG_K(1) TACG_K(2) TACG_K(3) TACG_K(4) TACG_K(5) TACG_K(6) TACG_K(7) TACG_K(8)
    TACG_K(9) TACG_K(10) TACG_K(11) TACG_K(12) TACG_K(13) TACG_K(14) TACG_K(15) TACG_K(16)
#undef TACG_K
    default:
      return false;
  }
}

int launch_eval_planes(const EvBase& e, const int64_t* fam_off_host, const int32_t* home_start_host,
                       const int32_t* home_size_host, hipStream_t stream) {
  PlArgs a{};
  a.trace = e.trace;
  a.primary = e.primary;
  a.ws = e.ws;
  a.N = e.N;
  a.L = e.L;
  a.E = e.E;
  a.F = e.F;
  a.G = e.G;
  a.P = e.P;
  int64_t tiles = 0;
  for (int f = 0; f < e.F; ++f) {
    const int64_t n = fam_off_host[f + 1] - fam_off_host[f];
    const int64_t hz = home_size_host[f];
    a.fam[f] = FamRec{static_cast<uint32_t>(fam_off_host[f]), static_cast<uint32_t>(fam_off_host[f + 1]),
                      static_cast<uint32_t>(tiles),
                      static_cast<uint32_t>(home_start_host[f]) | (static_cast<uint32_t>(hz) << 8)};
    tiles += ((n + hz - 1) / hz + 63) / 64 * hz;
  }
  for (int f = e.F; f <= TACG_MAX_FAMILIES; ++f) a.fam[f] = FamRec{0u, 0u, 0xffffffffu, 1u << 8};
  if (tiles == 0) return TACG_OK;
  if (tiles >= 0xffffffffll) return TACG_E_UNSUPPORTED;
  // placement blocks: 16 groups each, the rest in one block padded to a power of two (a block of 2^b groups steps 64 / 2^b
  // tokens at once).  Every block prepares all tokens and builds its own tables, so splitting the rest into smaller powers of
  // two only pays where few layers or tiles leave the chip idle (then a remainder of up to three quarters of a power of
  // two is split).  Whole calls, split / padded: E = 65, top-8, 64 families, 24 layers, 65 placements 102 / 70 us at 8 tokens a
  // family, 183 / 127 at 400; E = 128, top-8, 48 layers x 65536 tokens 300 / 213 at 65, 534 / 492 at 340, 745 / 769 at 577; E = 256, top-8,
  // 20 layers x 65536 633 / 468 at 700; but E = 100, top-10, 4 layers x 6000 tokens 68 / 87 at 384, E = 60, 2 layers x 120007 70 / 82.
  const bool full = e.L >= 16 && tiles * e.L >= 768;
  const int groups = (e.P + 31) / 32;
  a.n_full = groups / kCols;
  a.n_pblocks = a.n_full;
  for (int at = a.n_full * kCols, rest = groups % kCols; rest > 0;) {
    int sz = 1;
    while (sz < rest) sz *= 2;
    if (sz != rest && 4 * rest <= 3 * sz && !full) sz /= 2;
    a.tail[a.n_pblocks - a.n_full] = static_cast<uint32_t>(at) | (static_cast<uint32_t>(sz) << 24);
    ++a.n_pblocks;
    at += sz;
    rest -= std::min(sz, rest);
  }
  a.n_tiles = static_cast<uint32_t>(tiles);
  a.n_shares = static_cast<int32_t>(shares_of(tiles, static_cast<int64_t>(e.L) * a.n_pblocks, std::min(groups, kCols)));
  switch (e.K) {
#define TACG_K(k) \
  case k:         \
    return e.G <= 4 ? launch_t<k, 4>(a, stream) : launch_t<k, 8>(a, stream);
    TACG_K(1) TACG_K(2) TACG_K(3) TACG_K(4) TACG_K(5) TACG_K(6) TACG_K(7) TACG_K(8)
    TACG_K(9) TACG_K(10) TACG_K(11) TACG_K(12) TACG_K(13) TACG_K(14) TACG_K(15) TACG_K(16)
#undef TACG_K
    default:
      return TACG_E_UNSUPPORTED;
  }
}

}  // namespace tacg
