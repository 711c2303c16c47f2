// AllGather-GEMM, one rank's share (paper, Appendix "AllGather GEMM").
//
// One launch holds both roles.  The first `num_producers` work-groups are the emulated
// peers: shard by shard, in delivery order, they copy shard s into rows
// [s*m_per_rank, (s+1)*m_per_rank) of the workspace and then raise flag s (the copy is
// fused into the kernel rather than issued as separate memcpy calls).  Every other
// work-group is one output tile of the consumer GEMM: it maps its index to a tile through
// the chiplet remap, the grouped order and the rank rotation, waits for the flags of the
// shards its rows touch, and only then reads the workspace.  Producer work-groups have the
// lowest indices, so they are dispatched before any consumer can occupy a compute unit.
#include "gemm_core.h"
#include "launch.h"

namespace ditron {

struct AgGemmParams {
  const void* shard[DITRON_MAX_WORLD];
  int order[DITRON_MAX_WORLD];
  char* workspace;
  const char* b;
  __bf16* c;
  int32_t* flags;      // [world]
  int32_t* arrivals;   // [world] producer arrival counters
  int32_t* status;
  int32_t* schedule;   // or null
  int timing;          // schedule records hold time stamps instead
  const float* a_scales;   // fp8: one per shard, or null
  const float* b_scales;   // fp8: one per output column, or null
  int32_t* epoch_word;     // fp8, if set: the call's epoch is 1 + this word, which the last work-group to finish advances
  int32_t* finished;       // ... counting the work-groups that are done
  int m_per_rank, m, n, k, world, rank, nnodes;
  int32_t epoch;
  int num_producers, teams;
  unsigned spin_limit;
  int wait;            // 0: every shard is resident, the flags are not looked at
  TileOrder tiling;
};

// Scales of an fp8 tile: one per shard (rows), one per column.
struct ShardScales {
  const AgGemmParams& p;
  int m0, n0;
  __device__ __forceinline__ float row(int r) const { return p.a_scales ? p.a_scales[min(m0 + r, p.m - 1) / p.m_per_rank] : 1.f; }
  __device__ __forceinline__ f32x4_t cols(int c) const {   // n is a multiple of 8: the four columns are inside or none is
    if (!p.b_scales || n0 + c >= p.n) return f32x4_t{1.f, 1.f, 1.f, 1.f};
    const float* s = p.b_scales + n0 + c;
    return f32x4_t{s[0], s[1], s[2], s[3]};
  }
};

template <class T, bool ROTATE>
__device__ __forceinline__ void ag_gemm_work_group(const AgGemmParams& p, const int32_t epoch, char* lds) {
  constexpr int kElement = T::F8 ? 1 : 2;
  if ((int)blockIdx.x < p.num_producers) {
    const size_t shard_bytes = (size_t)p.m_per_rank * p.k * kElement;
    produce_chunks<T::THREADS>(
        p.world, shard_bytes, blockIdx.x, p.num_producers, p.teams, epoch,
        [&](int i) { return (void*)(p.workspace + (size_t)p.order[i] * shard_bytes); },
        [&](int i) { return p.shard[p.order[i]]; }, [&](int i) { return p.flags + p.order[i]; },
        [&](int i) { return p.arrivals + p.order[i]; });
    return;
  }
  const int wg = blockIdx.x - p.num_producers;
  const TileSpan t = tile_of_workgroup(wg, p.tiling, kOrderGather, p.m, p.m_per_rank, p.rank, p.world, p.nnodes, T::BM);
  const int m0 = t.pid_m * T::BM, n0 = t.pid_n * T::BN;
  const unsigned long long ts_start = p.timing ? wall_clock64() : 0;
  if (p.schedule && !p.timing && threadIdx.x == 0) {
    int32_t* rec = p.schedule + 4 * (size_t)wg;
    rec[0] = t.pid_m; rec[1] = t.pid_n; rec[2] = t.first; rec[3] = t.last;
  }
  if (p.wait) flag_wait_block(p.flags, t.first, t.last - t.first + 1, epoch, p.spin_limit, p.status);
  const unsigned long long ts_ready = p.timing ? wall_clock64() : 0;

  const uint32_t row_bytes = (uint32_t)p.k * kElement;
  const int M = p.m, N = p.n;
  auto a_row = [=](int r) { return (uint32_t)min(m0 + r, M - 1) * row_bytes; };
  typename T::Acc acc;
  if constexpr (T::B_KN) {
    gemm_mainloop<T>(acc, p.workspace, a_row, p.b, BColumns{(uint32_t)N * 2u, n0, N}, p.k, lds);
  } else {
    auto b_row = [=](int r) { return (uint32_t)min(n0 + r, N - 1) * row_bytes; };
    gemm_mainloop<T, ROTATE>(acc, p.workspace, a_row, p.b, b_row, T::F8 ? p.k / 2 : p.k, lds, ROTATE ? chiplet_k_tile(p.k) : 0);
  }
  if constexpr (T::F8) park_tile_bf16<T>(acc, lds, ShardScales{p, m0, n0});
  else park_tile_bf16<T>(acc, lds);
  store_parked_bf16<T>(p.c, (size_t)p.n, m0, n0, m0, M, N, lds);
  if (p.timing && threadIdx.x == 0) {
    int32_t* rec = p.schedule + 4 * (size_t)wg;
    rec[0] = (int32_t)(ts_start & 0x7fffffff); rec[1] = rec[0];
    rec[2] = (int32_t)(ts_ready & 0x7fffffff); rec[3] = (int32_t)(wall_clock64() & 0x7fffffff);
  }
}

// ROTATE: the K loop begins at chiplet_k_tile (a kernel of its own: both loops in one cost the plain one up to 1.5 %)
template <class T, bool ROTATE>
__global__ __launch_bounds__(T::THREADS) void ag_gemm_kernel(const AgGemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  if constexpr (T::F8) {
    // (the fp8 operator can be recorded and replayed at every size: see ag_gemm_splitk_kernel)
    const int32_t epoch = call_epoch(p.epoch, p.epoch_word);
    ag_gemm_work_group<T, ROTATE>(p, epoch, lds);
    advance_epoch(epoch, p.epoch_word, p.finished);
  } else {
    ag_gemm_work_group<T, ROTATE>(p, p.epoch, lds);
  }
}

template <class T, bool ROTATE = false>
static ditron_status_t launch_ag(AgGemmParams& p, hipStream_t stream) {
  p.tiling.npm = cdiv(p.m, T::BM);
  p.tiling.npn = cdiv(p.n, T::BN);
  if (!set_dynamic_lds<ag_gemm_kernel<T, ROTATE>>(T::LDS_BYTES)) return DITRON_ERR_HIP;
  const unsigned grid = (unsigned)(p.num_producers + p.tiling.npm * p.tiling.npn);
  hipLaunchKernelGGL((ag_gemm_kernel<T, ROTATE>), dim3(grid), dim3(T::THREADS), T::LDS_BYTES, stream, p);
  return hipGetLastError() == hipSuccess ? DITRON_OK : DITRON_ERR_HIP;
}

}  // namespace ditron

using namespace ditron;

extern "C" ditron_status_t ditron_ag_gemm(const void* const* a_shards, const void* b, int b_layout, void* c,
                                          const float* a_scales, const float* b_scales, void* workspace,
                                          int32_t* signals, int32_t* status, int32_t* schedule_out,
                                          const int* arrival_order, int m_per_rank, int n, int k, int world,
                                          int rank, int dtype, int32_t epoch, unsigned flags,
                                          const ditron_tuning_t* tuning, void* stream) {
  if (world < 1 || world > DITRON_MAX_WORLD || rank < 0 || rank >= world) return DITRON_ERR_INVALID_ARG;
  if (m_per_rank <= 0 || n <= 0 || k <= 0) return DITRON_ERR_INVALID_ARG;
  const Tuning tune = resolve_tuning(tuning, world);
  if (!tune.valid) return DITRON_ERR_INVALID_ARG;
  if (!b || !c || !workspace || !signals || !status) return DITRON_ERR_INVALID_ARG;
  if (!aligned16(b) || !aligned16(c) || !aligned16(workspace) || !aligned16(signals)) return DITRON_ERR_INVALID_ARG;
  const Mode mode = producer_mode(flags);
  if (mode == Mode::kInvalid) return DITRON_ERR_INVALID_ARG;
  const bool emulate = mode == Mode::kEmulate;
  if ((flags & (DITRON_DUMP_SCHEDULE | DITRON_DUMP_TIMING)) && !schedule_out) return DITRON_ERR_INVALID_ARG;
  if ((flags & DITRON_DUMP_SCHEDULE) && (flags & DITRON_DUMP_TIMING)) return DITRON_ERR_INVALID_ARG;
  if (b_layout != DITRON_B_KN && b_layout != DITRON_B_NK) return DITRON_ERR_INVALID_ARG;
  if (dtype != DITRON_BF16 && dtype != DITRON_FP8_E4M3) return DITRON_ERR_INVALID_ARG;
  if (emulate) {
    if (!a_shards) return DITRON_ERR_INVALID_ARG;
    for (int s = 0; s < world; ++s)
      if (!a_shards[s] || !aligned16(a_shards[s])) return DITRON_ERR_INVALID_ARG;
    if (arrival_order && !is_permutation(arrival_order, world)) return DITRON_ERR_INVALID_ARG;
  }
  const bool fp8 = dtype == DITRON_FP8_E4M3;
  const bool decode_shaped = ag_takes_decode_kernel(m_per_rank * world, n, k, dtype, b_layout, tune.decode_variant);
  if ((flags & DITRON_EPOCH_IN_MEMORY) && !decode_shaped && !fp8) return DITRON_ERR_UNSUPPORTED;
  if (decode_shaped)
    return ditron_ag_gemm_decode(a_shards, b, b_layout, c, a_scales, b_scales, workspace, signals, status, schedule_out,
                                 arrival_order, m_per_rank, n, k, world, rank, dtype, epoch, flags, tuning, stream);
  if (fp8 && b_layout != DITRON_B_NK) return DITRON_ERR_UNSUPPORTED;
  if (k % (fp8 ? 16 : 8) != 0 || n % 8 != 0) return DITRON_ERR_UNSUPPORTED;
  const int esize = fp8 ? 1 : 2;
  if (!fits_32bit((size_t)m_per_rank * world, k, esize) || !fits_32bit(n, k, esize)) return DITRON_ERR_UNSUPPORTED;

  AgGemmParams p{};
  for (int i = 0; i < world; ++i) {
    p.shard[i] = emulate ? a_shards[i] : nullptr;
    p.order[i] = arrival_order ? arrival_order[i] : (rank + i) % world;
  }
  p.workspace = (char*)workspace;
  p.b = (const char*)b;
  p.c = (__bf16*)c;
  p.flags = signals;
  p.arrivals = signals + world;
  p.status = status;
  p.schedule = (flags & (DITRON_DUMP_SCHEDULE | DITRON_DUMP_TIMING)) ? schedule_out : nullptr;
  p.timing = (flags & DITRON_DUMP_TIMING) != 0;
  p.m_per_rank = m_per_rank;
  p.m = m_per_rank * world;
  p.n = n;
  p.k = k;
  p.world = world;
  p.rank = rank;
  p.epoch = epoch;
  if (fp8) {
    p.a_scales = a_scales;
    p.b_scales = b_scales;
    if (flags & DITRON_EPOCH_IN_MEMORY) {
      const size_t words = ditron_signal_words(world, 1);
      p.epoch_word = signals + words - 1;
      p.finished = signals + words - 2;
    }
  }
  p.spin_limit = tune.spin_limit;
  p.wait = mode != Mode::kPreset;
  TileChoice tc = choose_tile(p.m, n, k, ag_narrow(dtype, b_layout));
  p.nnodes = nodes_of_order(p.m, tc.block_m, node_listing_rows(p.m, n, dtype), world, tune.num_nodes, rank, kOrderGather);
  if (!p.nnodes) return DITRON_ERR_UNSUPPORTED;
  p.tiling.group_m = tc.group_m;
  p.tiling.num_xcd = tc.num_xcd;
  p.tiling.per_xcd = tc.per_xcd;
  const ProducerPlan pl = plan_producers((size_t)p.m * k * esize, world, /*tiles_wait=*/true);
  p.num_producers = emulate ? pl.producers : 0;
  p.teams = pl.teams;
  if (b_layout == DITRON_B_KN) {
    if (tc.block_n == 224) return launch_ag<TileBigKN224>(p, (hipStream_t)stream);
    if (tc.block_n == 192) return launch_ag<TileBigKN192>(p, (hipStream_t)stream);
    if (tc.big) return launch_ag<TileBigKN>(p, (hipStream_t)stream);
    if (tc.block_n == 64) return launch_ag<TileSmallKN64>(p, (hipStream_t)stream);
    return launch_ag<TileSmallKN>(p, (hipStream_t)stream);
  }
  if (fp8) {
    if (tc.block_n == 224) return launch_ag<TileBigF8_224>(p, (hipStream_t)stream);
    if (tc.block_n == 192) return launch_ag<TileBigF8_192>(p, (hipStream_t)stream);
    return launch_ag<TileBigF8>(p, (hipStream_t)stream);
  }
  if (tc.big) {
    if (tc.block_n == 224) return launch_ag<TileBigDirect224>(p, (hipStream_t)stream);
    if (tc.block_n == 192) return launch_ag<TileBigDirect192>(p, (hipStream_t)stream);
    return launch_ag<TileBigDirect>(p, (hipStream_t)stream);
  }
  return rows_share_channels(k) ? launch_ag<TileSmall, true>(p, (hipStream_t)stream) : launch_ag<TileSmall>(p, (hipStream_t)stream);
}
