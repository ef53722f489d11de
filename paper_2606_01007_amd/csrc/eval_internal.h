// Declarations shared by the placement-scoring kernels (eval.hip, eval_planes.hip, eval_tokens.hip): the workspace layout and
// the arguments of the passes around the trace pass.
#pragma once

#include "tacg_internal.h"

namespace tacg {

constexpr uint8_t kNone = 0xFF;
constexpr int kMaxPieces = 160;
constexpr uint32_t kXcds = 8;  // XCDs of an MI355X; workgroups are dealt to them round-robin
struct EvWs {
  uint32_t* cnt;        // [L][E] dispatches per expert
  uint32_t* flagbits;   // [L][8] experts with a secondary in some placement
  uint8_t* rep_of;      // [L][E] compact replicated index or 0xFF
  int32_t* rep_list;    // [L][TACG_MAX_REPLICATED]
  int32_t* n_rep;       // [L]
  uint2* rep_info;      // [L][TACG_MAX_REPLICATED][P]  (FC mask, fallback GPU)
  // accumulators are laid out with the placement fastest, so that a workgroup's adds for its run of
  // placements are contiguous (coalesced atomics)
  unsigned long long* acc_home;  // [P]
  unsigned long long* acc_span;  // [P]
  unsigned long long* acc_fam;   // [F][P]
  uint32_t* rep_load;   // [L][G][P2], P2 = P rounded up to even: placement pairs share a 64-bit add
  // App. C statistics (used only by tacg_eval_trace_stats)
  uint32_t* cnt_fam;                  // [F][L][E] dispatches per expert and family
  unsigned long long* acc_span_fam;   // [F][P] sum of |cards| over the family's token-layers
  unsigned long long* acc_cross_fam;  // [F][P] token-layers whose cards span several bands
  unsigned long long* acc_hmass_fam;  // [F][P] replicated-slot dispatches served in the family's band
  unsigned long long* n_bad;          // [1] token-layers not scored: an id out of range or repeated
  uint32_t* bad_tiles;                // [ceil(N L / 64 / 32)] bit g: token-layers 64 g .. 64 g + 63 of
                                      // the flattened trace (x = l N + t) hold an invalid one
};

__host__ __device__ inline int32_t even_up(int32_t P) { return P + (P & 1); }

__host__ __device__ inline int64_t bad_tile_words(int64_t N, int32_t L) { return (N * L + 2047) / 2048; }

inline EvWs carve_ev(void* ws, int64_t N, int32_t L, int32_t E, int32_t G, int32_t P, int32_t F, size_t* used = nullptr) {
  Carver c{static_cast<char*>(ws), 0};
  EvWs r;
  r.cnt = c.take<uint32_t>(static_cast<size_t>(L) * E);
  r.flagbits = c.take<uint32_t>(static_cast<size_t>(L) * 8);
  r.acc_home = c.take<unsigned long long>(static_cast<size_t>(P));
  r.acc_span = c.take<unsigned long long>(static_cast<size_t>(P));
  r.acc_fam = c.take<unsigned long long>(static_cast<size_t>(P) * F);
  r.rep_load = c.take<uint32_t>(static_cast<size_t>(even_up(P)) * L * G);
  r.rep_of = c.take<uint8_t>(static_cast<size_t>(L) * E);
  r.rep_list = c.take<int32_t>(static_cast<size_t>(L) * TACG_MAX_REPLICATED);
  r.n_rep = c.take<int32_t>(static_cast<size_t>(L));
  r.rep_info = c.take<uint2>(static_cast<size_t>(L) * TACG_MAX_REPLICATED * P);
  r.cnt_fam = c.take<uint32_t>(static_cast<size_t>(F) * L * E);
  r.acc_span_fam = c.take<unsigned long long>(static_cast<size_t>(P) * F);
  r.acc_cross_fam = c.take<unsigned long long>(static_cast<size_t>(P) * F);
  r.acc_hmass_fam = c.take<unsigned long long>(static_cast<size_t>(P) * F);
  r.n_bad = c.take<unsigned long long>(1);
  r.bad_tiles = c.take<uint32_t>(static_cast<size_t>(bad_tile_words(N, L)));
  if (used) *used = c.used;
  return r;
}

// Arguments of the passes around the trace pass (small: they are copied at every launch) ...
struct EvBase {
  const int16_t* trace;
  const uint8_t* primary;
  const uint8_t* secondary;
  const int64_t* load_ref;
  uint32_t* d_err;
  EvWs ws;
  int64_t N;
  int32_t L, K, E, F, G, P, R;
  int32_t theta_num, theta_den;
  int32_t stats;      // App. C statistics requested
  uint32_t band_starts;  // bit b: a family band starts at GPU b (the bands tile 0..G-1)
};

// ... and of ev_main and ev_stats.
struct EvArgs : EvBase {
  int32_t n_pieces;
  int32_t n_pblocks;  // placement blocks of 64 * PPL placements
  // home band of family f: component f % 4 of band4[f / 4] = home_start | home_size << 8
  uint4 band4[TACG_MAX_FAMILIES / 4];
  // One record per piece of one family's tokens: (first token, end token, family offset,
  // home_start | home_size << 8 | family << 16).  Kept as 16-byte records: indexing kernel-argument
  // arrays of different element sizes with one runtime index lets the compiler fold the byte and
  // dword offsets into an unaligned scalar-load base, which the scalar unit does not honour.
  uint4 piece[kMaxPieces];
};
static_assert(sizeof(EvArgs) <= 4096, "kernel arguments must stay within 4 KB");

// The K int16 ids of a token-layer, fetched with the widest loads their alignment allows.
template <int K>
struct TraceIds {
  static constexpr int kWords = K % 2 == 0 ? K / 2 : K;
  uint32_t w[kWords];
  __device__ __forceinline__ void fetch(const int16_t* p) {
    if constexpr (K % 8 == 0) {
#pragma unroll
      for (int q = 0; q < K / 8; ++q) {
        const uint4 v = reinterpret_cast<const uint4*>(p)[q];
        w[4 * q] = v.x;
        w[4 * q + 1] = v.y;
        w[4 * q + 2] = v.z;
        w[4 * q + 3] = v.w;
      }
    } else if constexpr (K % 4 == 0) {
#pragma unroll
      for (int q = 0; q < K / 4; ++q) {
        const uint2 v = reinterpret_cast<const uint2*>(p)[q];
        w[2 * q] = v.x;
        w[2 * q + 1] = v.y;
      }
    } else if constexpr (K % 2 == 0) {
#pragma unroll
      for (int q = 0; q < K / 2; ++q) w[q] = reinterpret_cast<const uint32_t*>(p)[q];
    } else {
#pragma unroll
      for (int s = 0; s < K; ++s) w[s] = static_cast<uint16_t>(p[s]);
    }
  }
  __device__ __forceinline__ void unpack(uint32_t (&raw)[K]) const {
#pragma unroll
    for (int s = 0; s < K; ++s) raw[s] = K % 2 == 0 ? (w[s / 2] >> (16 * (s & 1))) & 0xffffu : w[K % 2 == 0 ? 0 : s];
  }
};

// The bit-plane trace pass (eval_planes.hip): whether it takes these sizes, and its launch.
bool eval_uses_planes(int32_t top_k, int32_t n_experts, int32_t n_gpus, int32_t n_sec, int64_t n_tokens,
                      int32_t families_with_tokens);
int launch_eval_planes(const EvBase& e, const int64_t* fam_off_host, const int32_t* home_start_host,
                       const int32_t* home_size_host, hipStream_t stream);

// The lane = token trace pass (eval_tokens.hip), also with the App. C statistics, and the numbers of placements it is
// taken for.  Its time grows with the placements, the other passes' hardly do.  Measured on MI355X per call (top-8, 2^17
// tokens x 16 layers), lane = token against lane = placement: E = 256, 32 GPUs, 16 x 3 replicas 204 / 312 us at 24
// placements, 242 / 312 at 32, 358 / 309 at 48; E = 128, 16 GPUs, no replicas 126 / 188 us at 48, 135 / 190 at 64 (above
// that the crossing depends on the sizes: at 96 to 128 placements 0.3 to 2.0 times lane = placement); against
// bit planes (E = 128, 8 GPUs, 8 x 2 replicas) 63 / 84 us at 4, 86 / 85 at 8, 137 / 89 at 16.
//
// A workgroup of lane = token scores four placements of one family's chunk, so from more than 24 placements on the set-up of
// its many workgroups (about 8.5 ns of the full chip each, against 50 ns for one of lane = placement) needs token-layers
// to pay for it, unless two rounds of workgroups hold them all (four with secondaries).  64 families, lane = token against lane = placement:
// E = 96, top-2, 64 placements, 58 layers x 356 tokens a family 550 / 185 us; E = 65, top-12, 32 placements, 24 layers x 10
// tokens 152 / 63 us; E = 64, top-6, 40 placements, 24 layers x 687 tokens 151 / 210 us; E = 192, top-16, 40 placements, 8 layers
// x 1612 tokens 173 / 307 us; 24 placements at most 19 / 18 us at any length.
inline bool eval_uses_tokens(int32_t n_place, int32_t n_sec, bool planes, int64_t n_tokens, int32_t n_layers, int32_t top_k,
                             int32_t families_with_tokens) {
  if (n_place > (planes ? 6 : n_sec > 0 ? 40 : 64)) return false;
  const int64_t fam = families_with_tokens > 0 ? families_with_tokens : 1;
  return n_place <= 24 || (n_place + 3) / 4 * fam * n_layers <= (n_sec > 0 ? 4096 : 2048) || n_tokens / fam * top_k >= 4096;
}
int launch_eval_tokens(const EvBase& e, const int64_t* fam_off_host, const int32_t* home_start_host,
                       const int32_t* home_size_host, hipStream_t stream);

}  // namespace tacg
