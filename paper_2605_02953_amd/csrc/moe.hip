// MoE AllGather + grouped GEMM, one rank's share (paper: "ag_group_gemm" of the kernel
// list; tile ordering after `threadblock_swizzle_ag_moe_kernel`, Appendix "Swizzle").
//
// Launch 1.  The first work-groups (integer only, up to eight sharing the scan plus one for the
// schedule): per-(rank, expert) histogram, exclusive scan of the local experts' totals, stable
// gather index, then the tile list: every local expert's rows are cut into BLOCK_M row tiles, each
// tile learns the span of source ranks its rows come from and the ring stage at which the last of
// them arrives, and tiles are emitted grouped by expert, ascending stage, ties in original order.
// The other work-groups are the emulated peers: they copy the token shards into the workspace in
// delivery order and raise one flag per shard.  The all-gather does not depend on the routing, so
// it starts with the call and runs beside the routing work-groups (which leave the rest of the chip idle).
// Launch 2: every work-group takes one (tile, column block), gathers its rows through gather_idx while
// staging them in LDS and multiplies by its expert's weights.  It waits for the shard flags of its tile if
// an external producer delivers the shards; emulated peers have delivered with launch 1.
#include "gemm_core.h"
#include "launch.h"
#include "reduce.h"

namespace ditron {

constexpr int kRouteThreads = 1024;
constexpr int kRouteWaves = kRouteThreads / 64;
constexpr int kMaxExperts = 256;       // experts (global) the routing kernel can histogram
constexpr int kMaxLocalExperts = 64;
constexpr int kMaxTilesLds = 4096;     // tile stages kept in LDS by the schedule step
constexpr int kRouteGroupsMax = 8;     // work-groups that share the routing scan
// what a routing work-group hands to the others: its (rank, expert) histogram, its totals of the local
// experts, and the smallest flat index at which it met an id that names no expert
constexpr int kPartLocal = DITRON_MAX_WORLD * kMaxExperts;
constexpr int kPartBad = kPartLocal + kMaxLocalExperts;
constexpr int kRoutePartWords = kPartBad + 64;
static_assert(kRouteGroupsMax * kRoutePartWords * 4 == DITRON_MOE_ROUTE_SCRATCH_BYTES, "scratch size declared at the boundary");
constexpr int kNoBadId = 0x7fffffff;
constexpr int kWalkExperts = 16;       // up to this many local experts a work-group finds its expert by a scalar walk

struct MoeRouteParams {
  const int32_t* topk_ids;   // [tokens * top_k]
  int32_t* counts;           // [world * num_experts]
  int32_t* expert_offsets;   // [num_local + 1]
  int32_t* gather_idx;       // [max_rows]
  int32_t* tile_records;     // [0] = ntiles ; 4 words per tile ; then max_tiles words: first row of the tile
  int32_t* status;
  int tokens_per_rank, top_k, num_experts, expert_begin, num_local, max_rows, max_tiles;
  int world, rank, block_m;
  // routing work-groups 0 .. groups-1 and the scheduling work-group `groups`
  int groups;
  int32_t* route_flags;      // [groups]
  int32_t* parts;            // [groups][kRoutePartWords]
  unsigned spin_limit;
  // the emulated peers (work-groups groups+1 .. groups+num_producers)
  const void* shard[DITRON_MAX_WORLD];
  int order[DITRON_MAX_WORLD];
  char* workspace;
  int32_t* flags;
  int32_t* arrivals;
  size_t shard_bytes;
  int32_t epoch;
  int num_producers, teams;
};

// Work-groups 0 .. G-1 share the scan of the assignments: each owns one contiguous range, cut into one
// contiguous range per wave, so that positions inside an expert follow the flat assignment index whatever G
// is.  A work-group histograms its range, hands its partial tables to the others through memory (one flag
// per work-group, bounded wait), and then places its own assignments: the first output position of (work-
// group, wave, expert) is the expert's offset plus what the ranges before it hold of that expert.
// Work-group G sums the histograms and writes counts, offsets and the tile list.  All G + 1 have the lowest
// indices of the launch, so they are resident before anything else and the waits end.
__global__ __launch_bounds__(kRouteThreads) void moe_route_kernel(const MoeRouteParams p) {
  __shared__ int s_counts[DITRON_MAX_WORLD * kMaxExperts];       // [world][num_experts]
  __shared__ int s_offsets[kMaxLocalExperts + 1];
  __shared__ int s_wave_base[kRouteWaves][kMaxLocalExperts];     // running output position per (wave, expert)
  __shared__ int s_tile_acc[kMaxLocalExperts + 1];               // exclusive prefix of tiles per expert
  __shared__ int s_cum[kMaxLocalExperts][DITRON_MAX_WORLD];      // inclusive per-rank cumulative rows per expert
  __shared__ int s_total[kMaxLocalExperts], s_before[kMaxLocalExperts];
  __shared__ int s_stage[kMaxTilesLds];
  __shared__ int s_bad;                                          // smallest flat index holding an id outside [0, E)
  const int G = p.groups;
  if ((int)blockIdx.x > G) {
    // the STREAM form: the grouped GEMM that reads the workspace is a later launch
    produce_chunks<kRouteThreads, true>(
        p.world, p.shard_bytes, blockIdx.x - G - 1, p.num_producers, p.teams, p.epoch,
        [&](int i) { return (void*)(p.workspace + (size_t)p.order[i] * p.shard_bytes); },
        [&](int i) { return p.shard[p.order[i]]; }, [&](int i) { return p.flags + p.order[i]; },
        [&](int i) { return p.arrivals + p.order[i]; });
    return;
  }
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int F = p.world * p.tokens_per_rank * p.top_k;
  const int per_shard = p.tokens_per_rank * p.top_k;
  const int E = p.num_experts, EL = p.num_local, WE = p.world * E;

  if ((int)blockIdx.x == G) {
    // ---------------------------------------------------------------- counts, offsets, tile list
    flag_wait_block(p.route_flags, 0, G, p.epoch, p.spin_limit, p.status);
    for (int i = tid; i < WE; i += kRouteThreads) {
      int c = 0;
      for (int g = 0; g < G; ++g) c += p.parts[g * kRoutePartWords + i];
      s_counts[i] = c;
      p.counts[i] = c;
    }
    if (tid == 0) {
      int bad = kNoBadId;
      for (int g = 0; g < G; ++g) bad = min(bad, p.parts[g * kRoutePartWords + kPartBad]);
      s_bad = bad;
    }
    __syncthreads();
    if (s_bad != kNoBadId) {
      // an id that names no expert: reported, never dropped silently (the counts would no longer sum to
      // tokens * top_k); no tile is scheduled
      if (tid == 0) {
        p.status[0] = DITRON_ERR_INVALID_ARG;
        p.status[1] = s_bad;
        p.tile_records[0] = 0;
      }
      return;
    }
    // per-rank cumulative rows of the local experts; exclusive scan of their totals
    if (tid < EL) {
      int run = 0;
      for (int s = 0; s < p.world; ++s) {
        run += s_counts[s * E + p.expert_begin + tid];
        s_cum[tid][s] = run;
      }
    }
    __syncthreads();
    if (tid == 0) {
      int run = 0, tiles = 0;
      for (int j = 0; j < EL; ++j) {
        s_offsets[j] = run;
        s_tile_acc[j] = tiles;
        const int n_j = s_cum[j][p.world - 1];
        run += n_j;
        tiles += cdiv(n_j, p.block_m);
      }
      s_offsets[EL] = run;
      s_tile_acc[EL] = tiles;
    }
    __syncthreads();
    for (int j = tid; j <= EL; j += kRouteThreads) p.expert_offsets[j] = s_offsets[j];
    const int R = s_offsets[EL];
    const int ntiles = s_tile_acc[EL];
    if (R > p.max_rows || ntiles > p.max_tiles || ntiles > kMaxTilesLds) {
      if (tid == 0) {
        p.status[0] = DITRON_ERR_WORKSPACE;
        p.status[2] = R;
        p.tile_records[0] = 0;
      }
      return;
    }
    // stage of a tile: position in the ring order rank, rank+1, ... of the last source rank among its rows
    for (int t = tid; t < ntiles; t += kRouteThreads) {
      int j = 0;
      while (s_tile_acc[j + 1] <= t) ++j;
      const int q0 = (t - s_tile_acc[j]) * p.block_m;
      const int q1 = min(q0 + p.block_m, s_cum[j][p.world - 1]);
      int seg_start = 0, seg_end = 0;
      for (int s = 0; s < p.world; ++s) {
        seg_start += (s_cum[j][s] <= q0);
        seg_end += (s_cum[j][s] <= q1 - 1);
      }
      int stage = 0;
      for (int s = seg_start; s <= seg_end; ++s) stage = max(stage, (s - p.rank + p.world) % p.world);
      s_stage[t] = stage | (seg_start << 8) | (seg_end << 16);
    }
    __syncthreads();
    int32_t* rec = p.tile_records + 1;
    int32_t* row0 = p.tile_records + 1 + 4 * p.max_tiles;
    for (int t = tid; t < ntiles; t += kRouteThreads) {
      int j = 0;
      while (s_tile_acc[j + 1] <= t) ++j;
      const int mine = s_stage[t] & 0xFF;
      int before = 0;
      for (int u = s_tile_acc[j]; u < s_tile_acc[j + 1]; ++u) {
        const int other = s_stage[u] & 0xFF;
        before += (other < mine) || (other == mine && u < t);
      }
      const int pos = s_tile_acc[j] + before;
      rec[4 * pos + 0] = j;
      rec[4 * pos + 1] = t;
      rec[4 * pos + 2] = (s_stage[t] >> 8) & 0xFF;
      rec[4 * pos + 3] = (s_stage[t] >> 16) & 0xFF;
      row0[pos] = s_offsets[j] + (t - s_tile_acc[j]) * p.block_m;
    }
    if (tid == 0) p.tile_records[0] = ntiles;
    return;
  }

  // ------------------------------------------------------------------ routing work-group g
  const int g = blockIdx.x;
  for (int i = tid; i < WE; i += kRouteThreads) s_counts[i] = 0;
  for (int i = tid; i < kRouteWaves * kMaxLocalExperts; i += kRouteThreads) (&s_wave_base[0][0])[i] = 0;
  if (tid == 0) s_bad = kNoBadId;
  __syncthreads();

  // histogram over (source rank, expert), and per-wave totals for the local experts.  The ids are fetched
  // kBatch steps at a time so that the loads overlap instead of queueing one by one.
  constexpr int kBatch = 16;
  const int per_wave = cdiv(cdiv(F, G * kRouteWaves), 64) * 64;
  const int w_begin = (int)min((long)(g * kRouteWaves + wave) * per_wave, (long)F), w_end = min(w_begin + per_wave, F);
  for (int f0 = w_begin; f0 < w_end; f0 += 64 * kBatch) {
    int e[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int f = f0 + b * 64 + lane;
      e[b] = f < w_end ? p.topk_ids[f] : -1;
    }
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int f = f0 + b * 64 + lane;
      if (f >= w_end) continue;
      if (e[b] >= 0 && e[b] < E) {
        atomicAdd(&s_counts[(f / per_shard) * E + e[b]], 1);
        const int j = e[b] - p.expert_begin;
        if (j >= 0 && j < EL) atomicAdd(&s_wave_base[wave][j], 1);
      } else {
        atomicMin(&s_bad, f);
      }
    }
  }
  __syncthreads();
  int32_t* part = p.parts + g * kRoutePartWords;
  for (int i = tid; i < WE; i += kRouteThreads) part[i] = s_counts[i];
  if (tid < EL) {
    int c = 0;
    for (int w = 0; w < kRouteWaves; ++w) c += s_wave_base[w][tid];
    part[kPartLocal + tid] = c;
  }
  if (tid == 0) part[kPartBad] = s_bad;
  __syncthreads();
  if (tid == 0) flag_raise(p.route_flags + g, p.epoch);
  flag_wait_block(p.route_flags, 0, G, p.epoch, p.spin_limit, p.status);

  // every routing work-group takes the same decisions from the same tables
  if (tid < EL) {
    int total = 0, before = 0;
    for (int h = 0; h < G; ++h) {
      const int c = p.parts[h * kRoutePartWords + kPartLocal + tid];
      total += c;
      before += h < g ? c : 0;
    }
    s_total[tid] = total;
    s_before[tid] = before;
  }
  if (tid == 64) {
    int bad = kNoBadId;
    for (int h = 0; h < G; ++h) bad = min(bad, p.parts[h * kRoutePartWords + kPartBad]);
    s_bad = bad;
  }
  __syncthreads();
  if (s_bad != kNoBadId) return;
  if (tid == 0) {
    int run = 0, tiles = 0;
    for (int j = 0; j < EL; ++j) {
      s_offsets[j] = run;
      run += s_total[j];
      tiles += cdiv(s_total[j], p.block_m);
    }
    s_offsets[EL] = run;
    s_tile_acc[EL] = tiles;
  }
  __syncthreads();
  if (s_offsets[EL] > p.max_rows || s_tile_acc[EL] > p.max_tiles || s_tile_acc[EL] > kMaxTilesLds) return;

  // first output position of every (wave, expert) of this work-group
  if (tid < EL) {
    int run = s_offsets[tid] + s_before[tid];
    for (int w = 0; w < kRouteWaves; ++w) {
      const int c = s_wave_base[w][tid];
      s_wave_base[w][tid] = run;
      run += c;
    }
  }
  __syncthreads();

  // stable placement: 64 assignments at a time.  The lanes that hold the same local expert find
  // each other with one ballot per bit of the expert index (a lane keeps the lanes that agree with
  // it on every bit) and rank themselves by counting the lanes below them.  The first lane of each
  // group moves the wave's running output position of that expert past the group with one LDS atomic,
  // whose return value is the group's first position; the others receive it by a lane shuffle.  The
  // row of running positions is private to the wave and a wave's LDS atomics execute in order, so
  // consecutive rounds see each other's advances.  The cost per round does not grow with the number
  // of local experts beyond the number of index bits.
  const int nbits = EL > 1 ? 32 - __builtin_clz(EL - 1) : 0;
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int fb = w_begin; fb < w_end; fb += 64 * kBatch) {
    int jj[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int f = fb + b * 64 + lane;
      int j = -1;
      if (f < w_end) {
        j = p.topk_ids[f] - p.expert_begin;
        if (j < 0 || j >= EL) j = -1;
      }
      jj[b] = j;
    }
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int f = fb + b * 64 + lane;
      const int j = jj[b];
      const bool local = j >= 0;
      unsigned long long same = __ballot(local);
      if (same == 0) continue;
      for (int bit = 0; bit < nbits; ++bit) {
        const bool set = local && ((j >> bit) & 1);
        const unsigned long long m = __ballot(set);
        same &= set ? m : ~m;
      }
      const int rank = __popcll(same & below), count = __popcll(same);
      int base = 0;
      if (local && rank == 0) base = atomicAdd(&s_wave_base[wave][j], count);
      base = __shfl(base, local ? __ffsll((long long)same) - 1 : lane);
      // (the range test only matters after a timed-out wait, when the tables may be incomplete)
      if (local && (unsigned)(base + rank) < (unsigned)p.max_rows) p.gather_idx[base + rank] = f;
    }
  }
}

struct MoeGemmParams {
  const char* workspace;
  const char* w;
  __bf16* y;
  const int32_t* expert_offsets;
  const int32_t* gather_idx;
  const int32_t* tile_records;   // null: expert after expert, cut into row tiles from expert_offsets, no arrival stage (every row is local)
  const int32_t* flags;
  int32_t* status;
  int max_rows;   // without tile_records: what expert_offsets may name at most
  int tokens_per_rank, hidden, inter, top_k, world, max_tiles, npn, num_local, num_xcd;   // hidden: contraction length, inter: output width
  int rows_in_place;   // 1: row p of the left operand is row p of `workspace` (already grouped by expert), no gather
  int32_t* inverse_idx;   // if set: the work-groups of column block 0 also write inverse_idx[gather_idx[p]] = p for their rows
  int assignments;
  int32_t epoch;
  unsigned spin_limit;
  int wait;   // 0: the token shards are resident, the flags are not looked at
};

// NST > 0: operands through a ring of NST LDS stages filled by four extra waves (expert weights stream from
// HBM: see gemm_mainloop_ring_split)
// WALK: the launch has fewer work-groups than items and every work-group walks down its chiplet's run with the
// stride of the grid (short tiles: a work-group start costs as much as the tile).
template <class T, int NST = 0, bool WALK = false>
__global__ __launch_bounds__(NST > 0 ? 2 * T::THREADS : T::THREADS) void moe_grouped_gemm_kernel(const MoeGemmParams p) {
  static_assert(!WALK || NST == 0, "the loading waves of the ring leave the kernel after one item");
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  // Work-group -> (row tile, column block).  All (row tile, column block) items are put in one list, expert
  // after expert, inside an expert column block after column block, the expert's row tiles (one to three) of
  // a column block next to each other; the list is cut into as many equal runs as there are chiplets and
  // chiplet x (the work-groups with index = x mod 8) takes run x.  Neighbours in the list share a block of the
  // expert's weights (same column block) or the gathered rows (same row tile), so each comes from memory about
  // once, and every chiplet has the same number of tiles (an expert per chiplet moves as few bytes but leaves
  // the chiplets of small experts idle while the large ones run two rounds).  The row tiles of expert j are
  // the positions [first_j, first_j + ceil(n_j / BLOCK_M)) of the tile list, in arrival-stage order.
  const int wg = blockIdx.x;
  const bool listed = p.tile_records != nullptr;
  int ntiles = 0;
  if (listed) {
    ntiles = p.tile_records[0];
    if (ntiles <= 0) return;   // nothing routed here, or the routing launch reported an error
  } else {
    const int rows = p.expert_offsets[p.num_local];
    if (rows > p.max_rows) {
      if (wg == 0 && threadIdx.x == 0) {
        p.status[0] = DITRON_ERR_WORKSPACE;
        p.status[2] = rows;
      }
      return;
    }
  }
  // lane j of every wave: the row tiles of expert j and of the experts before it (at most 64 local experts)
  const int lane_j = threadIdx.x & 63;
  int nt_j = 0, before_j = 0;
  if (WALK || !listed || p.num_local > kWalkExperts) {
    nt_j = lane_j < p.num_local ? cdiv(p.expert_offsets[lane_j + 1] - p.expert_offsets[lane_j], T::BM) : 0;
    before_j = nt_j;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int v = __shfl_up(before_j, d);
      if (lane_j >= d) before_j += v;
    }
    if (!listed) ntiles = __builtin_amdgcn_readlane(before_j, 63);
    before_j -= nt_j;
  }
  const int per_xcd = cdiv(ntiles * p.npn, p.num_xcd);
  const int slots_in_grid = WALK ? gridDim.x / p.num_xcd : per_xcd;
  for (int slot = wg / p.num_xcd; slot < per_xcd; slot += slots_in_grid) {
  const int item = (wg % p.num_xcd) * per_xcd + slot;
  if (item >= ntiles * p.npn) return;
  int nt, before, owner = 0;
  if (WALK || !listed || p.num_local > kWalkExperts) {
    // the expert whose items [before_j npn, (before_j + nt_j) npn) hold this one
    const unsigned long long holds = __ballot(item >= before_j * p.npn && item < (before_j + nt_j) * p.npn);
    if (holds == 0) return;
    owner = __ffsll((long long)holds) - 1;
    // (read into scalar registers: the tile's addresses derive from them and must stay wave-uniform)
    nt = __builtin_amdgcn_readlane(nt_j, owner);
    before = __builtin_amdgcn_readlane(before_j, owner);
  } else {
    // a handful of experts: a scalar walk over their offsets
    nt = 0;
    before = 0;
    for (int j = 0; j < p.num_local; ++j) {
      nt = cdiv(p.expert_offsets[j + 1] - p.expert_offsets[j], T::BM);
      if (item < (before + nt) * p.npn) break;
      before += nt;
    }
    if (nt == 0) return;
  }
  const int pid_n = (item - before * p.npn) / nt;
  const int pos = before + (item - before * p.npn) % nt;
  int j = owner, seg_start = 0, seg_end = 0, p0;
  if (listed) {
    const int32_t* rec = p.tile_records + 1 + 4 * pos;
    j = rec[0];
    seg_start = rec[2];
    seg_end = rec[3];
    p0 = p.tile_records[1 + 4 * p.max_tiles + pos];
  } else {
    p0 = p.expert_offsets[owner] + (pos - before) * T::BM;
  }
  const int p_end = min(p0 + T::BM, p.expert_offsets[j + 1]);
  if (p.wait) flag_wait_block(p.flags, seg_start, seg_end - seg_start + 1, p.epoch, p.spin_limit, p.status);
  if (p.inverse_idx && pid_n == 0) {
    // every row belongs to exactly one row tile, and every row tile has one work-group of column block 0
    for (int row = p0 + (int)threadIdx.x; row < p_end; row += (int)blockDim.x) {
      const int f = p.gather_idx[row];
      if (f >= 0 && f < p.assignments) p.inverse_idx[f] = row;
    }
  }

  const int n0 = pid_n * T::BN;
  const uint32_t row_bytes = (uint32_t)p.hidden * 2u;
  const char* wj = p.w + (size_t)j * p.inter * row_bytes;
  const int32_t* gidx = p.gather_idx;
  const int top_k = p.top_k, N = p.inter;
  // the gather happens here: a tile row is fetched from the token its assignment belongs to
  const int in_place = p.rows_in_place;
  auto a_row = [=](int r) {
    const int row = min(p0 + r, p_end - 1);
    return (uint32_t)(in_place ? row : gidx[row] / top_k) * row_bytes;
  };
  typename T::Acc acc;
  if constexpr (T::B_KN) {   // expert weights stored [hidden, inter]: same bytes per expert, inter contiguous
    gemm_mainloop<T>(acc, p.workspace, a_row, wj, BColumns{(uint32_t)N * 2u, n0, N}, p.hidden, lds);
  } else {
    auto b_row = [=](int r) { return (uint32_t)min(n0 + r, N - 1) * row_bytes; };
    if constexpr (NST > 0) {
      if (!gemm_mainloop_ring_split<T, NST>(acc, p.workspace, a_row, wj, b_row, p.hidden, lds)) {
        __syncthreads();   // the loading waves meet the barrier at the head of the epilogue and leave
        return;
      }
    } else {
      // (both loops in one kernel, unlike ag_gemm_kernel: the plain one takes the same time with the other one beside it, 8192 tokens, hidden
      // 4096, 8 of 64 experts 86.8, 86.9 us; 1024 tokens, 32 experts 65.3, 65.4; 256 tokens, hidden 7168, 8 experts 77.2, 77.3)
      constexpr bool kRotates = T::X16 && T::BM == 128;
      if (kRotates && rows_share_channels(p.hidden)) gemm_mainloop<T, kRotates>(acc, p.workspace, a_row, wj, b_row, p.hidden, lds, chiplet_k_tile(p.hidden));
      else gemm_mainloop<T>(acc, p.workspace, a_row, wj, b_row, p.hidden, lds);
    }
  }
  store_tile_bf16<T>(acc, p.y, (size_t)p.inter, p0, n0, p_end, N, lds);
  if constexpr (!WALK) return;
  __syncthreads();   // the parked tile has been read: the stages are idle for the next item
  }
}

}  // namespace ditron

using namespace ditron;


extern "C" int ditron_moe_max_tiles(int max_rows, int num_local_experts) {
  if (max_rows < 0 || num_local_experts < 0) return 0;
  return cdiv(max_rows, kMoeBlockM) + num_local_experts;
}

template <class T, int NST = 0>
static ditron_status_t launch_moe_gemm(MoeGemmParams& g, int max_tiles, hipStream_t s) {
  g.npn = cdiv(g.inter, T::BN);
  constexpr int kLds = NST > 0 ? NST * T::STAGE_BYTES : T::LDS_BYTES;
  static_assert(kLds <= 160 * 1024, "LDS of one compute unit");
  if (!set_dynamic_lds<moe_grouped_gemm_kernel<T, NST>>(kLds)) return DITRON_ERR_HIP;
  // every chiplet takes an equal share of the (row tile, column block) items
  const unsigned grid = (unsigned)(g.num_xcd * cdiv(max_tiles * g.npn, g.num_xcd));
  hipLaunchKernelGGL((moe_grouped_gemm_kernel<T, NST>), dim3(grid), dim3(NST > 0 ? 2 * T::THREADS : T::THREADS), kLds, s, g);
  return hipGetLastError() == hipSuccess ? DITRON_OK : DITRON_ERR_HIP;
}

// The same with at most `resident` work-groups, which share the items.
template <class T>
static ditron_status_t launch_moe_gemm_walk(MoeGemmParams& g, int max_tiles, int resident, hipStream_t s) {
  g.npn = cdiv(g.inter, T::BN);
  if (!set_dynamic_lds<moe_grouped_gemm_kernel<T, 0, true>>(T::LDS_BYTES)) return DITRON_ERR_HIP;
  const unsigned items = (unsigned)(g.num_xcd * cdiv(max_tiles * g.npn, g.num_xcd));
  const unsigned grid = std::min(items, (unsigned)(g.num_xcd * cdiv(resident, g.num_xcd)));
  hipLaunchKernelGGL((moe_grouped_gemm_kernel<T, 0, true>), dim3(grid), dim3(T::THREADS), T::LDS_BYTES, s, g);
  return hipGetLastError() == hipSuccess ? DITRON_OK : DITRON_ERR_HIP;
}

// 128-row tiles of [n, k] weights.  Their operands are streamed (an expert's weights are read by one or two row tiles).
// 128 columns: the 16 x 16 x 32 loop with three K tiles in flight.  192 and 256: a ring of as many LDS stages as fit (four and
// three), filled by waves of their own: the 16 x 16 x 32 loop has room for two K tiles of these widths only.  us for the whole call,
// weights not in the caches, with the ring and with that loop, 256 columns: 2048 tokens, hidden 4096, 64 experts top-6, 200 columns
// 85, 97; 256 columns 91, 100; 6000 tokens, 32 experts top-2, 512 columns 107, 113; hidden 2048, 2048 tokens top-4 75, 77.
// 128 columns: 8192 tokens, hidden 4096, 8 of 64 experts 91.1, 91.7; 1024 tokens, hidden 8192, 32 experts 121.6, 121.3, the same,
// and with the weights in the caches 1024 tokens, hidden 4096, 8 of 64 experts 52.4, 50.1.
static ditron_status_t launch_moe_gemm_128_rows(MoeGemmParams& g, int block_n, int max_tiles, hipStream_t s) {
  switch (block_n) {
    case 128: return launch_moe_gemm<GemmTile4W<128, 128, false, true, true>>(g, max_tiles, s);
    case 192: return launch_moe_gemm<GemmTile4W<128, 192, false, true>, 4>(g, max_tiles, s);
    default: return launch_moe_gemm<GemmTile4W<128, 256, false, true>, 3>(g, max_tiles, s);
  }
}

// The same for [k, n] weights.
static ditron_status_t launch_moe_gemm_256_rows_kn(MoeGemmParams& g, int block_n, int max_tiles, hipStream_t s) {
  if (block_n == 128) return launch_moe_gemm<GemmTile4W<256, 128, true, true, true>>(g, max_tiles, s);
  return launch_moe_gemm<TileBigKN>(g, max_tiles, s);
}
static ditron_status_t launch_moe_gemm_128_rows_kn(MoeGemmParams& g, int block_n, int max_tiles, hipStream_t s) {
  switch (block_n) {
    case 128: return launch_moe_gemm<TileSmallKN>(g, max_tiles, s);
    case 192: return launch_moe_gemm<GemmTile4W<128, 192, true, true, true>>(g, max_tiles, s);
    default: return launch_moe_gemm<GemmTile4W<128, 256, true, true, true>>(g, max_tiles, s);
  }
}

extern "C" ditron_status_t ditron_moe_ag_grouped_gemm(
    const void* const* x_shards, const int32_t* topk_ids, const void* w, int w_layout, void* y, int32_t* counts,
    int32_t* expert_offsets, int32_t* gather_idx, int32_t* tile_records, void* workspace, int32_t* signals,
    int32_t* status, const int* arrival_order, int tokens_per_rank, int hidden, int inter, int num_experts,
    int top_k, int expert_begin, int num_local_experts, int max_rows, int world, int rank, int32_t epoch,
    unsigned flags, const ditron_tuning_t* tuning, void* stream) {
  if (world < 1 || world > DITRON_MAX_WORLD || rank < 0 || rank >= world) return DITRON_ERR_INVALID_ARG;
  if (tokens_per_rank <= 0 || hidden <= 0 || inter <= 0 || num_experts <= 0 || top_k <= 0 || max_rows <= 0)
    return DITRON_ERR_INVALID_ARG;
  if (expert_begin < 0 || num_local_experts <= 0 || expert_begin + num_local_experts > num_experts)
    return DITRON_ERR_INVALID_ARG;
  if (!topk_ids || !w || !y || !counts || !expert_offsets || !gather_idx || !tile_records || !workspace ||
      !signals || !status)
    return DITRON_ERR_INVALID_ARG;
  if (!aligned16(w) || !aligned16(y) || !aligned16(workspace) || !aligned16(signals)) return DITRON_ERR_INVALID_ARG;
  const Mode mode = producer_mode(flags);
  if (flags & DITRON_EPOCH_IN_MEMORY) return DITRON_ERR_UNSUPPORTED;
  const Tuning tune = resolve_tuning(tuning, 1);
  if (mode == Mode::kInvalid || !tune.valid) return DITRON_ERR_INVALID_ARG;
  const bool emulate = mode == Mode::kEmulate;
  if (w_layout != DITRON_B_KN && w_layout != DITRON_B_NK) return DITRON_ERR_INVALID_ARG;
  if (emulate) {
    if (!x_shards) return DITRON_ERR_INVALID_ARG;
    for (int s = 0; s < world; ++s)
      if (!x_shards[s] || !aligned16(x_shards[s])) return DITRON_ERR_INVALID_ARG;
    if (arrival_order && !is_permutation(arrival_order, world)) return DITRON_ERR_INVALID_ARG;
  }
  if (hidden % 8 != 0 || inter % 8 != 0) return DITRON_ERR_UNSUPPORTED;
  if (!fits_32bit((size_t)world * tokens_per_rank, hidden, 2) || !fits_32bit(inter, hidden, 2))
    return DITRON_ERR_UNSUPPORTED;
  if (num_experts > kMaxExperts || num_local_experts > kMaxLocalExperts) return DITRON_ERR_UNSUPPORTED;
  if ((long)world * num_experts > (long)DITRON_MAX_WORLD * kMaxExperts) return DITRON_ERR_UNSUPPORTED;
  const int max_tiles = ditron_moe_max_tiles(max_rows, num_local_experts);
  if (max_tiles > kMaxTilesLds) return DITRON_ERR_UNSUPPORTED;
  if ((long)world * tokens_per_rank * top_k > 0x7fffffffL) return DITRON_ERR_UNSUPPORTED;

  hipStream_t s = (hipStream_t)stream;
  MoeRouteParams r{};
  r.topk_ids = topk_ids;
  r.counts = counts;
  r.expert_offsets = expert_offsets;
  r.gather_idx = gather_idx;
  r.tile_records = tile_records;
  r.status = status;
  r.tokens_per_rank = tokens_per_rank;
  r.top_k = top_k;
  r.num_experts = num_experts;
  r.expert_begin = expert_begin;
  r.num_local = num_local_experts;
  r.max_rows = max_rows;
  r.max_tiles = max_tiles;
  r.world = world;
  r.rank = rank;
  const long expected_rows = moe_expected_rows((long)world * tokens_per_rank, top_k, num_experts, num_local_experts);
  const MoeTile mt = choose_moe_tile(expected_rows, num_local_experts, inter);
  r.block_m = mt.block_m;
  for (int i = 0; i < world; ++i) {
    r.shard[i] = emulate ? x_shards[i] : nullptr;
    r.order[i] = arrival_order ? arrival_order[i] : (rank + i) % world;
  }
  r.workspace = (char*)workspace;
  r.flags = signals;
  r.arrivals = signals + world;
  // one routing work-group per 4096 assignments (three or four rounds of 64 per wave), eight at most
  const long assignments = (long)world * tokens_per_rank * top_k;
  r.groups = tune.moe_route_groups ? tune.moe_route_groups : (int)std::min<long>(kRouteGroupsMax, std::max<long>(1, assignments / 4096));
  r.route_flags = signals + 4 * world;   // behind the flags and counters of a one-chunk layout
  r.parts = (int32_t*)((char*)workspace + align256((size_t)world * tokens_per_rank * hidden * 2));
  r.spin_limit = tune.spin_limit;
  r.shard_bytes = (size_t)tokens_per_rank * hidden * 2;
  r.epoch = epoch;
  // as many work-groups (of 1024 threads here) as the plan for 256-thread producers: measured best of
  // a quarter, half, the same and twice as many (159, 127, 105, 125 us for the whole cfg 4 step)
  const ProducerPlan pl = plan_producers((size_t)world * r.shard_bytes, world);
  r.num_producers = emulate ? pl.producers : 0;
  r.teams = std::min(pl.teams, std::max(1, r.num_producers));
  hipLaunchKernelGGL(moe_route_kernel, dim3(r.groups + 1 + r.num_producers), dim3(kRouteThreads), 0, s, r);
  if (hipGetLastError() != hipSuccess) return DITRON_ERR_HIP;

  MoeGemmParams g{};
  g.workspace = (const char*)workspace;
  g.w = (const char*)w;
  g.y = (__bf16*)y;
  g.expert_offsets = expert_offsets;
  g.gather_idx = gather_idx;
  g.tile_records = tile_records;
  g.flags = signals;
  g.status = status;
  g.tokens_per_rank = tokens_per_rank;
  g.hidden = hidden;
  g.inter = inter;
  g.top_k = top_k;
  g.world = world;
  g.max_tiles = max_tiles;
  g.num_local = num_local_experts;
  g.num_xcd = 8;
  g.epoch = epoch;
  g.spin_limit = tune.spin_limit;
  g.wait = mode == Mode::kExternal;   // the emulated peers were work-groups of the launch before
  if (w_layout == DITRON_B_KN) {   // weights stored [hidden, inter]
    if (mt.block_m == 256)
      return launch_moe_gemm_256_rows_kn(g, moe_block_n_kn_256(expected_rows, num_local_experts, inter, mt.block_n), max_tiles, s);
    return launch_moe_gemm_128_rows_kn(g, moe_block_n_kn(expected_rows, num_local_experts, inter, mt.block_n), max_tiles, s);
  }
  if (mt.block_m == 256) {
    if (mt.block_n == 128) return launch_moe_gemm<GemmTile4W<256, 128>>(g, max_tiles, s);
    return launch_moe_gemm<TileBigDirect>(g, max_tiles, s);
  }
  return launch_moe_gemm_128_rows(g, mt.block_n, max_tiles, s);
}


// ====================================================================== MoE down-projection + ReduceScatter
// (paper: workload "MoE+ReduceScatter" of the evaluation; tensor-parallel placement.)  The activations are
// already grouped by expert (the output order of the AllGather + grouped GEMM above), so the grouped GEMM
// reads its rows in place; a top-k combine brings the rows back to token order (fp32 fma over the token's
// assignments in order, one rounding), and the reduce-scatter is the one of GEMM-ReduceScatter: the peers'
// blocks arrive in the scatter buffer, the slots are added in fp32 in slot order.
namespace ditron {

struct MoeCombineParams {
  const __bf16* y;             // [rows, hidden] grouped by expert
  int32_t* inverse_idx;        // [tokens * top_k]: where the grouped GEMM has put an assignment's row, or anything
  const int32_t* gather_idx;   // the assignment of a row
  const int32_t* expert_offsets;
  const float* gate;           // [tokens * top_k] or null
  __bf16* combined;            // [tokens, hidden]
  __bf16* out;                 // [tokens_per_rank, hidden] (moe_combine_sum_kernel)
  int tokens, tokens_per_rank, rank, world, top_k, hidden, num_local, max_rows, combine_wgs;
  // own-slot flags and the emulated peers (work-groups behind the combine)
  int32_t* done;               // work-groups of the combine that have finished the rank's own rows
  int32_t* own_flags;          // [chunks]
  const void* peer[DITRON_MAX_WORLD];
  int order[DITRON_MAX_WORLD];
  char* scatter_buf;
  int32_t* arr_flags;
  int32_t* arr_counters;
  size_t slot_bytes;
  int chunks, n_peers, num_producers, teams;
  int32_t epoch;
};

constexpr int kCombineThreads = 512;

// What a wave knows of a token's assignments, one lane each (at most 64 of them): the row, or -1 where the assignment's
// expert is not on this rank.  inverse_idx holds the row of every assignment that is here, and for the others whatever was there
// before, so a row counts only if it is the assignment's own (that takes a second load, and no launch that clears the index).
struct TokenRows {
  int f, row, owner;
  float gate;
  // assignments j0 .. j0 + 63 of token t (none if t < 0): first load and second load.  rows: how many there are
  __device__ __forceinline__ static TokenRows look_up(const MoeCombineParams& p, int t, int j0) {
    const int lane = threadIdx.x & 63;
    TokenRows r{-1, -1, -1, 1.f};
    if (t >= 0 && j0 + lane < p.top_k) {
      r.f = t * p.top_k + j0 + lane;
      r.row = p.inverse_idx[r.f];
      if (p.gate) r.gate = p.gate[r.f];
    }
    return r;
  }
  __device__ __forceinline__ void check(const MoeCombineParams& p, int rows) {
    if (row < 0 || row >= rows) row = -1;
    owner = row >= 0 ? p.gather_idx[row] : -1;
  }
};

// The combine and, behind it, the emulated peers; neither waits for anything.  (8192 tokens top-2 of 32 experts, 2048 columns, world
// 8: bound by memory, 101 MB for the combine itself, which take 17.6 us with the peers' blocks resident, and 59 MB for the peers' copies.)
// One wave per token and 64 U vectors of 8 columns, the rank's own rows first, U vectors of each of 8 / U of the token's rows in flight per
// lane; the last work-group to finish the own rows raises the flags of the own slot, for whoever waits on another stream.
template <int U>
__global__ __launch_bounds__(kCombineThreads) void moe_combine_kernel(const MoeCombineParams p) {
  if ((int)blockIdx.x >= p.combine_wgs) {
    const size_t chunk_bytes = p.slot_bytes / p.chunks;
    produce_chunks<kCombineThreads>(
        p.n_peers * p.chunks, chunk_bytes, blockIdx.x - p.combine_wgs, p.num_producers, p.teams, p.epoch,
        [&](int i) { return (void*)(p.scatter_buf + p.order[i / p.chunks] * p.slot_bytes + (i % p.chunks) * chunk_bytes); },
        [&](int i) { return (const void*)((const char*)p.peer[p.order[i / p.chunks]] + (i % p.chunks) * chunk_bytes); },
        [&](int i) { return p.arr_flags + p.order[i / p.chunks] * p.chunks + i % p.chunks; },
        [&](int i) { return p.arr_counters + p.order[i / p.chunks] * p.chunks + i % p.chunks; });
    return;
  }
  constexpr int kRows = 8 / U;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int vpr = p.hidden >> 3, blocks = cdiv(vpr, 64 * U);
  const int total_rows = p.expert_offsets[p.num_local];
  const int rows = total_rows > p.max_rows ? 0 : total_rows;   // too many: the grouped GEMM has reported it and written none
  const int stride = p.combine_wgs * (kCombineThreads / 64);
  const int own = p.tokens_per_rank * blocks, items = p.tokens * blocks;
  auto token_of = [&](int item) {
    const int t = p.rank * p.tokens_per_rank + item / blocks;
    return t >= p.tokens ? t - p.tokens : t;
  };
  auto look_up = [&](int item, int j0) { return TokenRows::look_up(p, item < items ? token_of(item) : -1, j0); };
  // through: the rows are written through (see stores_done), so that whoever is told of them needs no write-back
  auto run = [&](int first, int end, auto through) {
    TokenRows now = look_up(first, 0), next = look_up(first + stride, 0);
    now.check(p, rows);
    for (int item = first; item < end; item += stride) {
      TokenRows later = look_up(item + 2 * stride, 0);
      next.check(p, rows);
      const int t = token_of(item), block = item % blocks;
      float acc[U][8];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[u][q] = 0.f;
      for (int j0 = 0; j0 < p.top_k; j0 += 64) {
        if (j0 > 0) {
          now = look_up(item, j0);
          now.check(p, rows);
        }
        if (now.owner != now.f) now.row = -1;
        if (block == 0 && now.f >= 0 && now.row < 0) p.inverse_idx[now.f] = -1;
        const int n = min(64, p.top_k - j0);
        for (int j = 0; j < n; j += kRows) {
          // kRows rows of the token at a time, all their loads in flight together, then the sum in the order j = 0, 1, ...
          int row[kRows];
          float g[kRows];
          u32x4_t x[kRows][U];
#pragma unroll
          for (int b = 0; b < kRows; ++b) {
            row[b] = j + b < n ? __builtin_amdgcn_readlane(now.row, j + b) : -1;
            g[b] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, now.gate), min(j + b, n - 1)));
            if (row[b] >= 0) {
#pragma unroll
              for (int u = 0; u < U; ++u) {
                const int c = (block * U + u) * 64 + lane;
                if (c < vpr) x[b][u] = __builtin_nontemporal_load((const u32x4_t*)(p.y + (size_t)row[b] * p.hidden) + c);
              }
            }
          }
#pragma unroll
          for (int b = 0; b < kRows; ++b) {
            if (row[b] < 0) continue;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                acc[u][2 * q] = __builtin_fmaf(g[b], __builtin_bit_cast(float, x[b][u][q] << 16), acc[u][2 * q]);
                acc[u][2 * q + 1] = __builtin_fmaf(g[b], __builtin_bit_cast(float, x[b][u][q] & 0xFFFF0000u), acc[u][2 * q + 1]);
              }
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = (block * U + u) * 64 + lane;
        if constexpr (decltype(through)::value) {
          const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc((void*)(p.combined + (size_t)t * p.hidden), 0, p.hidden * 2, 0x00020000);
          __builtin_amdgcn_raw_buffer_store_b128(pack_bf16x8(acc[u]), out, c * 16, 0, kThrough);   // past the row nothing is written
        } else {
          if (c < vpr) *((u32x4_t*)(p.combined + (size_t)t * p.hidden) + c) = pack_bf16x8(acc[u]);
        }
      }
      now = next;
      next = later;
    }
  };
  const int first = blockIdx.x * (kCombineThreads / 64) + wave;
  // the last of the work-groups with rows of the rank's own to finish those raises the flags of the own slot
  const int own_wgs = min(p.combine_wgs, cdiv(own, kCombineThreads / 64));
  if ((int)blockIdx.x < own_wgs) {
    run(first, own, std::true_type{});
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) {
      const int old = __hip_atomic_fetch_add(p.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (old == own_wgs - 1) {
        __hip_atomic_store(p.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int c = 0; c < p.chunks; ++c) flag_raise_stored(p.own_flags + c, p.epoch);
      }
    }
  }
  run(first + cdiv(max(own - first, 0), stride) * stride, items, std::false_type{});
}

// The same where a wave takes 64 vectors of a token (few tokens or narrow rows), with the rest of the call in it: the lane that has combined
// a vector of the rank's own rows also delivers the peers' (unless they are resident) and adds the slots in their order.  A lane adds
// what it holds itself: nothing is waited for, neither flags nor other work-groups, and the launch of the reduction falls away.  The
// work-group that finishes own rows last raises the flags of the slots, for whoever waits on another stream.
// Such calls are bound by launches and round trips to memory: the peers' vectors are asked for before the token's rows are known, and the code is
// kept short (6.2 KB; with branches around loads 9 KB and 1 us more a call, with a second loop for the others' rows and the next item's vectors asked
// for ahead 18 KB and 2 to 3 us more).  us with the reduction behind the combine and with this kernel, top-2: 8 ranks, 7 tokens each of 1408 columns
// 14.1, 11.6; 16 of 3000 21.2, 19.7; 127 of 1024 19.0, 14.2; 1024 of 512 29.7, 23.4; 2 ranks, 33 of 2032 14.9, 12.3; 4096 of 512 36.0, 25.8;
// 8 ranks, top-6, 7 of 1392 20.9, 15.8; 512 of 128 20.2, 16.3.
__global__ __launch_bounds__(kCombineThreads) void moe_combine_sum_kernel(const MoeCombineParams p) {
  constexpr int kSlots = 8;   // slots in flight
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blocks = cdiv(p.hidden >> 3, 64);
  const int total_rows = p.expert_offsets[p.num_local];
  const int rows = total_rows > p.max_rows ? 0 : total_rows;   // too many: the grouped GEMM has reported it and written none
  const int own = p.tokens_per_rank * blocks, items = p.tokens * blocks, stride = p.combine_wgs * (kCombineThreads / 64);
  // one row of a block of rows, or nothing (no loads, no stores) where `exists` is false
  auto row_of = [&](const void* base, bool exists, int row) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)base + (size_t)row * p.hidden * 2, 0, exists ? p.hidden * 2 : 0, 0x00020000);
  };
  for (int item = blockIdx.x * (kCombineThreads / 64) + wave; item < items; item += stride) {
    const int r = item / blocks, block = item % blocks, vec = (block * 64 + lane) * 16;
    const int t = p.rank * p.tokens_per_rank + r < p.tokens ? p.rank * p.tokens_per_rank + r : p.rank * p.tokens_per_rank + r - p.tokens;
    const bool is_own = item < own;
    TokenRows now = TokenRows::look_up(p, t, 0);
    float sum[8];
    u32x4_t mine;
    for (int s0 = 0; s0 < (is_own ? p.world : 1); s0 += kSlots) {
      u32x4_t x[kSlots];
      if (is_own) {
#pragma unroll
        for (int b = 0; b < kSlots; ++b) {
          const int s = min(s0 + b, p.world - 1);
          const char* slot = p.peer[s] ? (const char*)p.peer[s] : p.scatter_buf + s * p.slot_bytes;
          x[b] = __builtin_amdgcn_raw_buffer_load_b128(row_of(slot, s0 + b < p.world && s != p.rank, r), vec, 0, kStreaming);
        }
      }
      if (s0 == 0) {
        now.check(p, rows);
        float acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.f;
        for (int j0 = 0; j0 < p.top_k; j0 += 64) {
          if (j0 > 0) {
            now = TokenRows::look_up(p, t, j0);
            now.check(p, rows);
          }
          if (now.owner != now.f) now.row = -1;
          if (block == 0 && now.f >= 0 && now.row < 0) p.inverse_idx[now.f] = -1;
          const int n = min(64, p.top_k - j0);
          for (int j = 0; j < n; j += kSlots) {
            // as in moe_combine_kernel; the loads of rows that are not there are of an empty buffer
            u32x4_t y[kSlots];
#pragma unroll
            for (int b = 0; b < kSlots; ++b) {
              const int row = j + b < n ? __builtin_amdgcn_readlane(now.row, min(j + b, 63)) : -1;
              y[b] = __builtin_amdgcn_raw_buffer_load_b128(row_of(p.y, row >= 0, max(row, 0)), vec, 0, kStreaming);
            }
#pragma unroll
            for (int b = 0; b < kSlots; ++b) {
              if (j + b >= n || __builtin_amdgcn_readlane(now.row, min(j + b, 63)) < 0) continue;
              const float g = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, now.gate), min(j + b, 63)));
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                acc[2 * q] = __builtin_fmaf(g, __builtin_bit_cast(float, y[b][q] << 16), acc[2 * q]);
                acc[2 * q + 1] = __builtin_fmaf(g, __builtin_bit_cast(float, y[b][q] & 0xFFFF0000u), acc[2 * q + 1]);
              }
            }
          }
        }
        mine = pack_bf16x8(acc);
        __builtin_amdgcn_raw_buffer_store_b128(mine, row_of(p.combined, true, t), vec, 0, kThrough);   // past the row nothing is written
      }
      if (is_own) {
#pragma unroll
        for (int b = 0; b < kSlots; ++b) {
          const int s = s0 + b;
          if (s < p.world) {
            __builtin_amdgcn_raw_buffer_store_b128(x[b], row_of(p.scatter_buf + s * p.slot_bytes, p.peer[s] != nullptr, r), vec, 0, kThrough);
            const u32x4_t term = s == p.rank ? mine : x[b];
            if (s == 0) set_bf16x8(sum, term);
            else add_bf16x8(sum, term);
          }
        }
      }
    }
    if (is_own) __builtin_amdgcn_raw_buffer_store_b128(pack_bf16x8(sum), row_of(p.out, true, r), vec, 0, kStreaming);
  }
  const int own_wgs = min(p.combine_wgs, cdiv(own, kCombineThreads / 64));
  if ((int)blockIdx.x >= own_wgs) return;
  stores_done();
  __syncthreads();
  if (threadIdx.x >= 64) return;
  int old = 0;
  if (lane == 0) old = __hip_atomic_fetch_add(p.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (__builtin_amdgcn_readfirstlane(old) != own_wgs - 1) return;
  if (lane == 0) __hip_atomic_store(p.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int i = lane; i < p.world * p.chunks; i += 64)
    if (i / p.chunks == p.rank || p.peer[i / p.chunks]) flag_raise_stored(p.arr_flags + i, p.epoch);
}

}  // namespace ditron

extern "C" ditron_status_t ditron_moe_grouped_gemm_rs(
    const void* h, const void* w, int w_layout, const float* topk_weights, const int32_t* gather_idx,
    const int32_t* expert_offsets, void* y, int32_t* inverse_idx, int32_t* tile_records, void* combined,
    const void* const* peer_partials, void* scatter_buf, void* out, int32_t* signals, int32_t* status,
    const int* arrival_order, int tokens_per_rank, int hidden, int inter, int num_experts, int top_k,
    int num_local_experts, int max_rows, int world, int rank, int chunks_per_slot, int32_t epoch, unsigned flags,
    const ditron_tuning_t* tuning, void* stream) {
  if (world < 1 || world > DITRON_MAX_WORLD || rank < 0 || rank >= world) return DITRON_ERR_INVALID_ARG;
  if (tokens_per_rank <= 0 || hidden <= 0 || inter <= 0 || num_experts <= 0 || top_k <= 0 || max_rows <= 0)
    return DITRON_ERR_INVALID_ARG;
  if (num_local_experts <= 0 || num_local_experts > num_experts || chunks_per_slot < 1 ||
      tokens_per_rank % chunks_per_slot != 0)
    return DITRON_ERR_INVALID_ARG;
  if (!h || !w || !gather_idx || !expert_offsets || !y || !inverse_idx || !tile_records || !combined || !out ||
      !signals || !status)
    return DITRON_ERR_INVALID_ARG;
  if (world > 1 && !scatter_buf) return DITRON_ERR_INVALID_ARG;
  if (!aligned16(h) || !aligned16(w) || !aligned16(y) || !aligned16(combined) || !aligned16(out) ||
      !aligned16(scatter_buf) || !aligned16(signals))
    return DITRON_ERR_INVALID_ARG;
  const Mode mode = producer_mode(flags);
  if (flags & DITRON_EPOCH_IN_MEMORY) return DITRON_ERR_UNSUPPORTED;
  const Tuning tune = resolve_tuning(tuning, 1);
  if (mode == Mode::kInvalid || !tune.valid) return DITRON_ERR_INVALID_ARG;
  const bool emulate = mode == Mode::kEmulate;
  if (w_layout != DITRON_B_KN && w_layout != DITRON_B_NK) return DITRON_ERR_INVALID_ARG;
  if (hidden % 8 != 0 || inter % 8 != 0) return DITRON_ERR_UNSUPPORTED;
  if (!fits_32bit((size_t)max_rows, inter, 2) || !fits_32bit(hidden, inter, 2)) return DITRON_ERR_UNSUPPORTED;
  if (num_local_experts > kMaxLocalExperts) return DITRON_ERR_UNSUPPORTED;
  const long assignments = (long)world * tokens_per_rank * top_k;
  if (assignments > 0x7fffffffL) return DITRON_ERR_UNSUPPORTED;
  const int max_tiles = ditron_moe_max_tiles(max_rows, num_local_experts);
  hipStream_t s = (hipStream_t)stream;

  int order[DITRON_MAX_WORLD] = {0};
  if (emulate && world > 1) {
    if (!peer_partials) return DITRON_ERR_INVALID_ARG;
    bool seen[DITRON_MAX_WORLD] = {false};
    for (int i = 0; i < world - 1; ++i) {
      const int sr = arrival_order ? arrival_order[i] : ((rank - 1 - i) % world + world) % world;
      if (sr < 0 || sr >= world || sr == rank || seen[sr]) return DITRON_ERR_INVALID_ARG;
      seen[sr] = true;
      order[i] = sr;
      if (!peer_partials[sr] || !aligned16(peer_partials[sr])) return DITRON_ERR_INVALID_ARG;
    }
  }

  // (tile_records is not needed: the grouped GEMM cuts its row tiles from expert_offsets)
  const long expected_rows = moe_expected_rows((long)world * tokens_per_rank, top_k, num_experts, num_local_experts);
  const MoeTile mt = choose_moe_tile(expected_rows, num_local_experts, hidden);

  // 1. grouped GEMM y[p, :] = h[p, :] . W2_expert(p): contraction over the intermediate size, hidden columns; its
  //    work-groups of column block 0 also write the inverse index of their rows
  MoeGemmParams g{};
  g.workspace = (const char*)h;
  g.w = (const char*)w;
  g.y = (__bf16*)y;
  g.expert_offsets = expert_offsets;
  g.gather_idx = gather_idx;
  g.tile_records = nullptr;
  g.max_rows = max_rows;
  g.flags = signals;
  g.status = status;
  g.tokens_per_rank = tokens_per_rank;
  g.hidden = inter;
  g.inter = hidden;
  g.top_k = top_k;
  g.world = world;
  g.max_tiles = max_tiles;
  g.num_local = num_local_experts;
  g.num_xcd = 8;
  g.rows_in_place = 1;
  g.inverse_idx = inverse_idx;
  g.assignments = (int)assignments;
  g.epoch = epoch;
  g.spin_limit = tune.spin_limit;
  g.wait = 0;
  ditron_status_t st;
  if (w_layout == DITRON_B_KN) {
    // Contractions of a few K tiles: 128 x 128 tiles with two K tiles in flight, which leave room for a second work-group on the
    // unit.  Longer ones: 256 columns where the tiles need several rounds.  us for the whole call, weights not in the caches, with these
    // tiles / 256 columns / 128 columns and three K tiles in flight: 64 tokens, 64 experts top-4, 6000 columns K 200 73 / 80 / 89, 512
    // 107 / 110 / 122, 768 137 / 139 / 152; 2048 tokens, 32 experts top-4, 2048 columns 200 73 / 75 / 78, 512 83.2 / 83.6 / 88, 1024
    // 106 / 103 / 108; 144 tokens, 8 experts top-6, 8064 columns 200 41.7 / 41.9 / 43.7, 512 47.5 / 47.0 / 49.7, 2000 86 / 77 / 87.
    if (mt.block_m == 256)
      st = launch_moe_gemm_256_rows_kn(g, moe_block_n_kn_256(expected_rows, num_local_experts, hidden, mt.block_n), max_tiles, s);
    else if (inter <= 512) st = launch_moe_gemm<TileSmallKNPaired>(g, max_tiles, s);
    else st = launch_moe_gemm_128_rows_kn(g, moe_block_n_kn(expected_rows, num_local_experts, hidden, 256), max_tiles, s);
  } else if (mt.block_m == 256) {
    st = mt.block_n == 128 ? launch_moe_gemm<GemmTile4W<256, 128>>(g, max_tiles, s) : launch_moe_gemm<TileBigDirect>(g, max_tiles, s);
  } else {
    // [n, k] weights and a contraction of a few K tiles: a tile is over before the ring of stages is full and costs about what a
    // work-group start costs, so 128 x 128 tiles on the two-stage loop (two work-groups fit a unit) and as many
    // work-groups as are resident at once, each walking down its share of the items (measured at the paper's
    // MoE+RS shape, whole call: 115 us with the ring tiles, 109 with these tiles, 106.5 with 512 resident
    // work-groups, 113.6 with 768; 256 x 256 tiles 108-118).
    st = inter <= 256 ? launch_moe_gemm_walk<TileSmallStaged>(g, max_tiles, 512, s)
                      : launch_moe_gemm_128_rows(g, mt.block_n, max_tiles, s);
  }
  if (st != DITRON_OK) return st;

  // 2. top-k combine into token order; the emulated peers' blocks arrive beside it, and where few items are all there is it sums as well
  const size_t slot_bytes = (size_t)tokens_per_rank * hidden * 2;
  MoeCombineParams c{};
  c.y = (const __bf16*)y;
  c.inverse_idx = inverse_idx;
  c.gather_idx = gather_idx;
  c.expert_offsets = expert_offsets;
  c.gate = topk_weights;
  c.combined = (__bf16*)combined;
  c.out = (__bf16*)out;
  c.tokens = world * tokens_per_rank;
  c.tokens_per_rank = tokens_per_rank;
  c.rank = rank;
  c.world = world;
  c.top_k = top_k;
  c.hidden = hidden;
  c.num_local = num_local_experts;
  c.max_rows = max_rows;
  const int vpr = hidden / 8;
  auto items_at = [&](int u) { return (long)c.tokens * cdiv(vpr, 64 * u); };
  // As many vectors per lane as leave a thousand waves; fewer tokens take more of a token's rows at a time instead, over more waves.  us
  // with 4, 2 and 1, whole calls (the reduction was part of the launch then): 8192 tokens top-2, 2048 columns 70, 73, 81; 1488 top-6, 1456 columns 42.3, 45.9, 50.1; 1200 top-1, 1072 columns
  // 21.5, 23.3, 24.2; 100 top-4, 1136 columns 22.1, 19.1, 17.5; 68 top-4, 7408 columns 42.0, 36.8, 36.2 (against: 2044 top-6, 2168 columns 64, 59, 54).
  const int unroll = vpr > 128 && items_at(4) >= 1024 ? 4 : vpr > 64 && items_at(2) >= 1024 ? 2 : 1;
  const long items = items_at(unroll);
  // three work-groups to a unit fit; 8192 tokens, 2048 columns, world 8: 256 / 512 / 768 of them 83 / 78 / 77 us for the call beside 56 copying
  // work-groups; 768 / 1024 68 / 73 beside 112
  c.combine_wgs = (int)std::min<long>(768, (items + kCombineThreads / 64 - 1) / (kCombineThreads / 64));
  c.done = signals + world;                                   // the counter word of segment 0 (unused here otherwise)
  c.own_flags = signals + 2 * world + rank * chunks_per_slot;
  for (int i = 0; i < world; ++i) {
    c.peer[i] = (emulate && i != rank && world > 1) ? peer_partials[i] : nullptr;
    c.order[i] = order[i];
  }
  c.scatter_buf = (char*)scatter_buf;
  c.arr_flags = signals + 2 * world;
  c.arr_counters = signals + 2 * world + world * chunks_per_slot;
  c.slot_bytes = slot_bytes;
  c.chunks = chunks_per_slot;
  c.n_peers = world - 1;
  const ProducerPlan pl = plan_producers((size_t)(world - 1) * slot_bytes, (world - 1) * chunks_per_slot);
  // twice as many as the plan says: they have half of its threads (at the same sizes 56 / 84 / 112 / 168 of them 77 / 72 / 68 / 68 us)
  c.num_producers = (emulate && world > 1) ? 2 * pl.producers : 0;
  c.teams = std::min(pl.teams, std::max(1, c.num_producers));
  c.epoch = epoch;
  if (unroll == 1 && mode != Mode::kExternal) {   // (an external producer's blocks are waited for by the reduction below)
    hipLaunchKernelGGL(moe_combine_sum_kernel, dim3((unsigned)c.combine_wgs), dim3(kCombineThreads), 0, s, c);
    return hipGetLastError() == hipSuccess ? DITRON_OK : DITRON_ERR_HIP;
  }
  const void* slots[DITRON_MAX_WORLD];
  for (int i = 0; i < world; ++i)
    slots[i] = i == rank ? (const void*)((const char*)combined + (size_t)rank * slot_bytes)
                         : (const void*)((const char*)scatter_buf + (size_t)i * slot_bytes);
  const dim3 grid((unsigned)(c.combine_wgs + c.num_producers));
  if (unroll == 4) hipLaunchKernelGGL(moe_combine_kernel<4>, grid, dim3(kCombineThreads), 0, s, c);
  else if (unroll == 2) hipLaunchKernelGGL(moe_combine_kernel<2>, grid, dim3(kCombineThreads), 0, s, c);
  else hipLaunchKernelGGL(moe_combine_kernel<1>, grid, dim3(kCombineThreads), 0, s, c);
  if (hipGetLastError() != hipSuccess) return DITRON_ERR_HIP;

  // 3. the reduction of GEMM-ReduceScatter over the `world` slots (own slot: the rank's rows of `combined`).  A launch of its own, so that
  //    the stream orders it and only an external producer's blocks are waited for.  As work-groups of the launch before, it held units while
  //    it polled for the combine, and preset flags told it nothing.  us in that launch and in its own: 8192 tokens, 2048 columns, world 8
  //    71.7, 67.5; 2044 tokens top-6, 2168 columns, 4 ranks 82.1, 68.5; 1024 tokens, 4096 columns, 2 ranks 68.9, 57.4; 1488 top-6,
  //    1456 columns 33.9, 34.9; 1200 top-1, 1072 columns 19.8, 20.2.
  return ditron_reduce_slots(slots, out, mode == Mode::kExternal ? signals + 2 * world : nullptr, status, tokens_per_rank, hidden, world,
                             chunks_per_slot, epoch, tuning, stream);
}
