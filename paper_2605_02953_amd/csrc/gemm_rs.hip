// GEMM-ReduceScatter, one rank's share (paper, Appendix "GEMM Reduce-Scatter").
//
// Launch 1 holds the GEMM and the emulated peers.  The last `num_producers` work-groups
// copy, peer by peer in delivery order and row chunk by row chunk, the block each peer would
// push into this rank's scatter buffer, raising one flag per (peer, chunk).  The first
// work-groups are the tiles of the local GEMM P = A . B, visited from the segment of rank+1
// to the rank's own segment; a tile bumps the counter of every segment it touches and the
// tile that completes a segment raises the segment flag.
// Launch 2 is the reduction: it adds the `world` blocks in fp32 in slot order with 128-bit loads and
// rounds once to bf16.  Only an external producer's flags are waited for (those of the row chunk that a
// work-group sums, and the GEMM's for the own segment); emulated peers have delivered with launch 1.
#include "gemm_core.h"
#include "launch.h"
#include "reduce.h"

namespace ditron {

struct GemmRsParams {
  const void* peer[DITRON_MAX_WORLD];
  int order[DITRON_MAX_WORLD];
  const char* a;
  const char* b;
  __bf16* gemm_out;
  __bf16* dst[DITRON_MAX_WORLD];   // fused scatter: rank d's [world, m_per_rank, n] buffer (dst[rank] is the local one)
  int fuse_scatter;
  char* scatter_buf;
  int32_t* seg_flags;      // [world]
  int32_t* seg_counters;   // [world]
  int32_t* arr_flags;      // [world * chunks]
  int32_t* arr_counters;   // [world * chunks]
  int32_t* status;
  int32_t* schedule;
  int m, n, k, world, rank, nnodes, m_per_rank, chunks, n_peers;
  int32_t epoch;
  int num_producers, teams;
  TileOrder tiling;
};

template <class T>
__global__ __launch_bounds__(T::THREADS) void gemm_rs_kernel(const GemmRsParams p) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int ntiles = p.tiling.npm * p.tiling.npn;
  if ((int)blockIdx.x >= ntiles) {
    // The emulated peers sit behind the GEMM tiles in the grid: nothing in this launch waits for
    // them (only the reduction does), so they fill compute units as the last tiles drain instead
    // of taking units away from the GEMM's first wave.
    const int part = blockIdx.x - ntiles;
    const size_t slot_bytes = (size_t)p.m_per_rank * p.n * 2;
    const size_t chunk_bytes = slot_bytes / p.chunks;
    // chunk index i = (delivery position of the peer) * chunks + row chunk
    produce_chunks<T::THREADS>(
        p.n_peers * p.chunks, chunk_bytes, part, p.num_producers, p.teams, p.epoch,
        [&](int i) { return (void*)(p.scatter_buf + p.order[i / p.chunks] * slot_bytes + (i % p.chunks) * chunk_bytes); },
        [&](int i) { return (const void*)((const char*)p.peer[p.order[i / p.chunks]] + (i % p.chunks) * chunk_bytes); },
        [&](int i) { return p.arr_flags + p.order[i / p.chunks] * p.chunks + i % p.chunks; },
        [&](int i) { return p.arr_counters + p.order[i / p.chunks] * p.chunks + i % p.chunks; });
    return;
  }
  const int wg = blockIdx.x;
  const TileSpan t = tile_of_workgroup(wg, p.tiling, kOrderScatter, p.m, p.m_per_rank, p.rank, p.world, p.nnodes, T::BM);
  const int m0 = t.pid_m * T::BM, n0 = t.pid_n * T::BN;
  const int seg_start = t.first, seg_end = t.last;
  if (p.schedule && threadIdx.x == 0) {
    int32_t* rec = p.schedule + 4 * (size_t)wg;
    rec[0] = t.pid_m; rec[1] = t.pid_n; rec[2] = seg_start; rec[3] = seg_end;
  }
  const uint32_t row_bytes = (uint32_t)p.k * 2u;
  const int M = p.m, N = p.n;
  auto a_row = [=](int r) { return (uint32_t)min(m0 + r, M - 1) * row_bytes; };
  typename T::Acc acc;
  if constexpr (T::B_KN) {
    gemm_mainloop<T>(acc, p.a, a_row, p.b, BColumns{(uint32_t)N * 2u, n0, N}, p.k, lds);
  } else {
    auto b_row = [=](int r) { return (uint32_t)min(n0 + r, N - 1) * row_bytes; };
    gemm_mainloop<T>(acc, p.a, a_row, p.b, b_row, p.k, lds);
  }
  // written through: the segment counter below announces the tile, and the partial is read only by the reduction, later
  if (p.fuse_scatter) {
    // the rows of segment d go straight to slot `rank` of rank d's buffer, row m landing at
    // rank * m_per_rank + m % m_per_rank (the listing's remote store)
    park_tile_bf16<T>(acc, lds);
    for (int seg = seg_start; seg <= seg_end; ++seg) {
      __bf16* c = p.dst[seg] + (ptrdiff_t)(p.rank - seg) * p.m_per_rank * p.n;
      store_parked_bf16<T, true>(c, (size_t)p.n, m0, n0, max(m0, seg * p.m_per_rank),
                                 min(min(m0 + T::BM, M), (seg + 1) * p.m_per_rank), N, lds);
    }
  } else {
    store_tile_bf16<T, true>(acc, p.gemm_out, (size_t)p.n, m0, n0, M, N, lds);
  }

  // segment completion: one lane per touched segment
  stores_done();
  __syncthreads();
  const int seg = seg_start + (int)threadIdx.x;
  if (seg <= seg_end) {
    const int first = (p.m_per_rank * seg) / T::BM;
    const int last = (p.m_per_rank * (seg + 1) - 1) / T::BM;
    const int target = p.tiling.npn * (last - first + 1);
    const int old = __hip_atomic_fetch_add(p.seg_counters + seg, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == target - 1) {
      __hip_atomic_store(p.seg_counters + seg, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      flag_raise_stored(p.seg_flags + seg, p.epoch);
    }
  }
}

// ------------------------------------------------------------------ reduction
struct ReduceParams {
  const void* slot[DITRON_MAX_WORLD];
  const int32_t* gate[DITRON_MAX_WORLD];  // first flag of slot s (chunk c at gate[s] + c*gate_stride[s]) or null
  int gate_stride[DITRON_MAX_WORLD];
  __bf16* out;
  int32_t* status;
  size_t vec_per_chunk;  // 16-byte vectors per row chunk
  int chunks, world;
  int32_t epoch;
  unsigned spin_limit;
  int wgs_per_chunk;
};

constexpr int kReduceThreads = 1024;
constexpr int kReduceMaxWgs = 1024;

// WORLD > 0 fixes the number of slots at compile time.  TOGETHER: a lane has a vector of every slot in flight before the first is added;
// otherwise one after another, and the other waves of the unit cover the wait: the chip's loads then walk the slots roughly in step, which
// the memory likes better.  us one after another and together, buffers not in the caches, 8 slots of 0.26 MB 6.9, 5.1; 2.1 MB 7.5, 6.1; 4.2 MB
// (256 work-groups) 8.8, 8.2; 6.3 MB 11.3, 11.3; 8.4 MB 13.1, 14.0; 16.8 MB 24.5, 26.9; 134 MB 198, 228; 4 slots of 4.2 MB 6.3, 6.0; 8.4 MB 8.2, 8.7;
// 134 MB 107, 118; 2 slots of 4.2 MB 5.1, 4.7; 134 MB 64.5, 67.3.
template <int WORLD, bool TOGETHER>
__global__ __launch_bounds__(kReduceThreads) void reduce_slots_kernel(const ReduceParams p) {
  const int chunk = blockIdx.x / p.wgs_per_chunk;
  const int part = blockIdx.x % p.wgs_per_chunk;
  const int world = WORLD > 0 ? WORLD : p.world;
  // one lane per slot: the flags are looked at side by side, not one round trip after another
  if ((int)threadIdx.x < world && p.gate[threadIdx.x])
    flag_wait_lane(p.gate[threadIdx.x], chunk * p.gate_stride[threadIdx.x], 1, p.epoch, p.spin_limit, p.status);
  __syncthreads();
  const size_t base = (size_t)chunk * p.vec_per_chunk;
  const size_t step = (size_t)p.wgs_per_chunk * kReduceThreads;
  u32x4_t* out = (u32x4_t*)p.out + base;
  for (size_t i = (size_t)part * kReduceThreads + threadIdx.x; i < p.vec_per_chunk; i += step) {
    float acc[8];
    if constexpr (WORLD > 0 && TOGETHER) {
      u32x4_t v[WORLD];
#pragma unroll
      for (int s = 0; s < WORLD; ++s) v[s] = __builtin_nontemporal_load((const u32x4_t*)p.slot[s] + base + i);
      set_bf16x8(acc, v[0]);
#pragma unroll
      for (int s = 1; s < WORLD; ++s) add_bf16x8(acc, v[s]);
    } else {
      set_bf16x8(acc, __builtin_nontemporal_load((const u32x4_t*)p.slot[0] + base + i));
#pragma unroll
      for (int s = 1; s < world; ++s) {
        __builtin_amdgcn_sched_barrier(0);   // (the compiler would put the loads together where it sees all of them)
        add_bf16x8(acc, __builtin_nontemporal_load((const u32x4_t*)p.slot[s] + base + i));
      }
    }
    __builtin_nontemporal_store(pack_bf16x8(acc), out + i);
  }
}

// `flags_pending`: some gate may still be down when the kernel starts (an external producer
// that needs room on the chip to run); the waiting work-groups are then kept to half the chip.
static ditron_status_t launch_reduce(ReduceParams& p, bool flags_pending, hipStream_t stream) {
  // enough work-groups to cover the chip several times over, at least one per row chunk
  size_t want = (p.vec_per_chunk + kReduceThreads - 1) / kReduceThreads;
  const int max_wgs = flags_pending ? 256 : kReduceMaxWgs;
  const size_t cap = (size_t)(max_wgs / p.chunks > 0 ? max_wgs / p.chunks : 1);
  if (want > cap) want = cap;
  if (want < 1) want = 1;
  p.wgs_per_chunk = (int)want;
  const dim3 grid((unsigned)(p.wgs_per_chunk * p.chunks));
  // up to a work-group per unit: 16 waves a unit are too few to cover a load of each slot in turn
  const bool together = grid.x <= 256;
  auto launch = [&](auto world) {
    constexpr int W = decltype(world)::value;
    if (together) hipLaunchKernelGGL((reduce_slots_kernel<W, true>), grid, dim3(kReduceThreads), 0, stream, p);
    else hipLaunchKernelGGL((reduce_slots_kernel<W, false>), grid, dim3(kReduceThreads), 0, stream, p);
  };
  switch (p.world) {
    case 8: launch(std::integral_constant<int, 8>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 2: launch(std::integral_constant<int, 2>{}); break;
    default: hipLaunchKernelGGL((reduce_slots_kernel<0, false>), grid, dim3(kReduceThreads), 0, stream, p); break;
  }
  return hipGetLastError() == hipSuccess ? DITRON_OK : DITRON_ERR_HIP;
}

template <class T>
static ditron_status_t launch_rs(GemmRsParams& p, hipStream_t stream) {
  p.tiling.npm = cdiv(p.m, T::BM);
  p.tiling.npn = cdiv(p.n, T::BN);
  if (!set_dynamic_lds<gemm_rs_kernel<T>>(T::LDS_BYTES)) return DITRON_ERR_HIP;
  const unsigned grid = (unsigned)(p.num_producers + p.tiling.npm * p.tiling.npn);
  hipLaunchKernelGGL(gemm_rs_kernel<T>, dim3(grid), dim3(T::THREADS), T::LDS_BYTES, stream, p);
  return hipGetLastError() == hipSuccess ? DITRON_OK : DITRON_ERR_HIP;
}

}  // namespace ditron

using namespace ditron;

extern "C" ditron_status_t ditron_reduce_slots(const void* const* slots, void* out, const int32_t* signals,
                                               int32_t* status, int rows, int n, int world, int chunks,
                                               int32_t epoch, const ditron_tuning_t* tuning, void* stream) {
  if (world < 1 || world > DITRON_MAX_WORLD || rows <= 0 || n <= 0 || chunks < 1) return DITRON_ERR_INVALID_ARG;
  const Tuning tune = resolve_tuning(tuning, 1);
  if (!tune.valid) return DITRON_ERR_INVALID_ARG;
  if (!slots || !out || !aligned16(out) || (signals && !status)) return DITRON_ERR_INVALID_ARG;
  if (n % 8 != 0) return DITRON_ERR_UNSUPPORTED;
  if (rows % chunks != 0) return DITRON_ERR_INVALID_ARG;
  ReduceParams p{};
  for (int s = 0; s < world; ++s) {
    if (!slots[s] || !aligned16(slots[s])) return DITRON_ERR_INVALID_ARG;
    p.slot[s] = slots[s];
    p.gate[s] = signals ? signals + (size_t)s * chunks : nullptr;
    p.gate_stride[s] = 1;
  }
  p.out = (__bf16*)out;
  p.status = status;
  p.vec_per_chunk = (size_t)(rows / chunks) * n / 8;
  p.chunks = chunks;
  p.world = world;
  p.epoch = epoch;
  p.spin_limit = tune.spin_limit;
  return launch_reduce(p, /*flags_pending=*/signals != nullptr, (hipStream_t)stream);
}

static ditron_status_t gemm_rs_impl(const void* a, const void* b, int b_layout, void* gemm_out,
                                    void* const* scatter_dsts, const void* const* peer_partials, void* scatter_buf,
                                    void* out, int32_t* signals, int32_t* status, int32_t* schedule_out,
                                    const int* arrival_order, int m, int n, int k_local, int world, int rank,
                                    int chunks_per_slot, int32_t epoch, unsigned flags,
                                    const ditron_tuning_t* tuning, void* stream) {
  const bool fuse = scatter_dsts != nullptr;

  if (world < 1 || world > DITRON_MAX_WORLD || rank < 0 || rank >= world) return DITRON_ERR_INVALID_ARG;
  if (m <= 0 || n <= 0 || k_local <= 0 || m % world != 0 || chunks_per_slot < 1) return DITRON_ERR_INVALID_ARG;
  const Tuning tune = resolve_tuning(tuning, world);
  if (!tune.valid) return DITRON_ERR_INVALID_ARG;
  const int m_r = m / world;
  if (m_r % chunks_per_slot != 0) return DITRON_ERR_INVALID_ARG;
  if (!a || !b || (!fuse && !gemm_out) || !out || !signals || !status) return DITRON_ERR_INVALID_ARG;
  if (world > 1 && !scatter_buf) return DITRON_ERR_INVALID_ARG;
  if (!aligned16(a) || !aligned16(b) || !aligned16(gemm_out) || !aligned16(out) || !aligned16(scatter_buf) ||
      !aligned16(signals))
    return DITRON_ERR_INVALID_ARG;
  const Mode mode = producer_mode(flags);
  if (flags & DITRON_EPOCH_IN_MEMORY) return DITRON_ERR_UNSUPPORTED;
  if (mode == Mode::kInvalid) return DITRON_ERR_INVALID_ARG;
  const bool emulate = mode == Mode::kEmulate;
  if ((flags & DITRON_DUMP_SCHEDULE) && !schedule_out) return DITRON_ERR_INVALID_ARG;
  if (b_layout != DITRON_B_KN && b_layout != DITRON_B_NK) return DITRON_ERR_INVALID_ARG;
  if (k_local % 8 != 0 || n % 8 != 0) return DITRON_ERR_UNSUPPORTED;
  if (!fits_32bit(m, k_local, 2) || !fits_32bit(n, k_local, 2)) return DITRON_ERR_UNSUPPORTED;

  GemmRsParams p{};
  p.n_peers = world - 1;
  if (emulate) {
    if (world > 1 && !peer_partials) return DITRON_ERR_INVALID_ARG;
    bool seen[DITRON_MAX_WORLD] = {false};
    for (int i = 0; i < world - 1; ++i) {
      const int s = arrival_order ? arrival_order[i] : ((rank - 1 - i) % world + world) % world;
      if (s < 0 || s >= world || s == rank || seen[s]) return DITRON_ERR_INVALID_ARG;
      seen[s] = true;
      p.order[i] = s;
      if (!peer_partials[s] || !aligned16(peer_partials[s])) return DITRON_ERR_INVALID_ARG;
      p.peer[s] = peer_partials[s];
    }
  }
  p.a = (const char*)a;
  p.b = (const char*)b;
  p.gemm_out = (__bf16*)gemm_out;
  p.fuse_scatter = fuse;
  if (fuse) {
    for (int d = 0; d < world; ++d) {
      if (!scatter_dsts[d] || !aligned16(scatter_dsts[d])) return DITRON_ERR_INVALID_ARG;
      p.dst[d] = (__bf16*)scatter_dsts[d];
    }
  }
  p.scatter_buf = (char*)scatter_buf;
  p.seg_flags = signals;
  p.seg_counters = signals + world;
  p.arr_flags = signals + 2 * world;
  p.arr_counters = signals + 2 * world + world * chunks_per_slot;
  p.status = status;
  p.schedule = (flags & DITRON_DUMP_SCHEDULE) ? schedule_out : nullptr;
  p.m = m;
  p.n = n;
  p.k = k_local;
  p.world = world;
  p.rank = rank;
  p.m_per_rank = m_r;
  p.chunks = chunks_per_slot;
  p.epoch = epoch;
  TileChoice tc = choose_tile(m, n, k_local, Narrow::kNever);
  p.nnodes = nodes_of_order(m, tc.block_m, node_listing_rows(m, n, DITRON_BF16), world, tune.num_nodes, rank, kOrderScatter);
  if (!p.nnodes) return DITRON_ERR_UNSUPPORTED;
  p.tiling.group_m = tc.group_m;
  p.tiling.num_xcd = tc.num_xcd;
  p.tiling.per_xcd = tc.per_xcd;
  const ProducerPlan pl = plan_producers((size_t)(world - 1) * m_r * n * 2, (world - 1) * chunks_per_slot);
  p.num_producers = (emulate && world > 1) ? pl.producers : 0;
  p.teams = pl.teams;
  // 128 x 128 tiles that fill the chip together with the peers' copies: two work-groups to a unit, so that the copies and the tiles
  // of a last, partly empty round run beside others.  us with one and with two to a unit, weights not in the caches, 8 ranks: 245
  // tiles + 16 copying work-groups, 640 x 6272, K 1024 41.2, 39.2; 1536 48.6, 44.2; 3584 65.5, 60.0 (2 ranks, 8 of them: all in one
  // round, 51.8, 59.6); 256 tiles, 2048 x 2048, 2048 47.8, 46.7; 3584 66.1, 57.2 ([k, n] 64.9, 56.8); 320, 2048 x 2560, 70.5, 64.2; 480, 1000 x
  // 7680, 83.1, 79.6; 240 + 16, 2048 x 1920, K 3584 49.4, 56.1.
  const int tiles = cdiv(m, 128) * cdiv(n, 128);
  const bool paired = tiles + p.num_producers > 256;
  ditron_status_t st;
  if (b_layout == DITRON_B_KN) {
    st = tc.big               ? launch_rs<TileBigKN>(p, (hipStream_t)stream)
         : tc.block_n == 64 ? launch_rs<TileSmallKN64>(p, (hipStream_t)stream)
         : paired           ? launch_rs<TileSmallKNPaired>(p, (hipStream_t)stream)
                            : launch_rs<TileSmallKN>(p, (hipStream_t)stream);
  } else {
    st = tc.big               ? launch_rs<TileBigDirect>(p, (hipStream_t)stream)
         : tc.block_n == 64 ? launch_rs<TileSmall64>(p, (hipStream_t)stream)
         : paired           ? launch_rs<TileSmallPaired>(p, (hipStream_t)stream)
                            : launch_rs<TileSmall>(p, (hipStream_t)stream);
  }
  if (st != DITRON_OK) return st;

  ReduceParams r{};
  const size_t slot_bytes = (size_t)m_r * n * 2;
  for (int s = 0; s < world; ++s) {
    if (s == rank) {
      r.slot[s] = fuse ? (const char*)scatter_buf + (size_t)rank * slot_bytes : (const char*)gemm_out + (size_t)rank * slot_bytes;
      r.gate[s] = mode == Mode::kExternal ? p.seg_flags + rank : nullptr;   // the GEMM's flag for the own segment gates every chunk
      r.gate_stride[s] = 0;
    } else {
      r.slot[s] = (const char*)scatter_buf + (size_t)s * slot_bytes;
      // otherwise the peers' blocks are resident, or the launch before this one has delivered them
      r.gate[s] = mode == Mode::kExternal ? p.arr_flags + (size_t)s * chunks_per_slot : nullptr;
      r.gate_stride[s] = 1;
    }
  }
  r.out = (__bf16*)out;
  r.status = status;
  r.vec_per_chunk = (size_t)(m_r / chunks_per_slot) * n / 8;
  r.chunks = chunks_per_slot;
  r.world = world;
  r.epoch = epoch;
  r.spin_limit = tune.spin_limit;
  // with emulated peers (or everything resident) every flag was raised by the launch before this one
  return launch_reduce(r, /*flags_pending=*/mode == Mode::kExternal, (hipStream_t)stream);
}

extern "C" ditron_status_t ditron_gemm_rs(const void* a, const void* b, int b_layout, void* gemm_out,
                                          const void* const* peer_partials, void* scatter_buf, void* out,
                                          int32_t* signals, int32_t* status, int32_t* schedule_out,
                                          const int* arrival_order, int m, int n, int k_local, int world, int rank,
                                          int chunks_per_slot, int32_t epoch, unsigned flags,
                                          const ditron_tuning_t* tuning, void* stream) {
  return gemm_rs_impl(a, b, b_layout, gemm_out, nullptr, peer_partials, scatter_buf, out, signals, status, schedule_out,
                      arrival_order, m, n, k_local, world, rank, chunks_per_slot, epoch, flags, tuning, stream);
}

extern "C" ditron_status_t ditron_gemm_rs_fuse_scatter(const void* a, const void* b, int b_layout,
                                                       void* const* scatter_dsts, const void* const* peer_partials,
                                                       void* out, int32_t* signals, int32_t* status,
                                                       int32_t* schedule_out, const int* arrival_order, int m, int n,
                                                       int k_local, int world, int rank, int chunks_per_slot,
                                                       int32_t epoch, unsigned flags,
                                                       const ditron_tuning_t* tuning, void* stream) {
  if (!scatter_dsts || world < 1 || world > DITRON_MAX_WORLD || rank < 0 || rank >= world) return DITRON_ERR_INVALID_ARG;
  return gemm_rs_impl(a, b, b_layout, nullptr, scatter_dsts, peer_partials, scatter_dsts[rank], out, signals, status,
                      schedule_out, arrival_order, m, n, k_local, world, rank, chunks_per_slot, epoch, flags, tuning,
                      stream);
}
