// GEMM + AllReduce in one-shot form, one rank's share (paper, Appendix "GEMM All-Reduce").
//
// One launch holds up to three kinds of work-groups.
//  * GEMM tiles: one work-group per tile of P = A . B, taken in the grouped tile order; it stores
//    the tile as bf16 into the buffer the peers would read and raises the tile's flag in this
//    rank's flag array.
//  * The emulated peers (lowest indices): every other rank's partial is resident in this GPU's
//    memory, so a peer is reduced to what the consumer sees of it, its tile flags, raised in the
//    order a peer's own GEMM finishes tiles.
//  * The sum.  One-shot with one tile per unit at most, or with nearly two (see launch_ar): the tile's
//    own work-group waits for the tile's flag of every peer and adds the peers' copies to its own, which it
//    still has in LDS.  It has published its tile before it waits, and every rank takes the tiles in the
//    same order, so the first tile that some rank has not published is always one that runs: no rank can block another.
//    Otherwise consumers: work-groups that draw tickets; ticket q is the tile at position q
//    of the tile order, so tiles are reduced in the order they are finished.  The holder waits
//    for the tile's flag of every rank (one lane per rank).  Either way the `world` published copies
//    are added in fp32 in rank order with 128-bit loads, rounded once to bf16 and written to the output tile.
// us with consumers and with the tiles' own sums, 8 ranks: 128 x 2048, K 512 (16 tiles) 16.6, 12.8; 64 x 4096, K 1024 15.2, 13.8; 16 x 8192, K 2048
// 17.7, 16.8; 512 x 8192, K 3584 (256 tiles) 45.6, 41.6; 4096 x 4096, K 2048 (256 large ones) 105.6, 103.2; 200 x 4096, K 1000, 2 ranks 16.3, 14.9.
// Two rounds (X as below; w: ranks):
//  * fewer than X units are left empty and t_gemm >= 3 t_reduce (large tiles: 3.5): 1024 x 8064 (504 tiles), K 3584 w2 84.0, 74.1; w4 87.1, 78.6; w8 93.1,
//    89.3; 512 w8 92.5, 92.2; 464 tiles, K 1536 w2 47.8, 43.8; K 2560 w4 71.2, 61.9; 512, K 1536 w2 45.9, 46.5; K 4096 w4 90.6, 90.0; 4608 x 7168
//    (504 large ones), K 3584 w2 239, 205; 512 large ones, K 2560 w4 187, 179;
//  * the same, t_gemm between that and 0.5 t_reduce: 512 tiles, K 2048 w8 65.5, 72.0; K 1024 w4 41.1, 43.7; 512 large ones, K 2048
//    w8 192, 206; w4 161, 163; K 3584 w8 266, 271; 504, K 2048 w8 186, 207;
//  * t_gemm below half of t_reduce: 512 tiles, K 512 w8 45.9, 52.6; K 256 w4 34.5, 34.5; 512 large ones, K 512 w8 152, 142; K 256 w8 140, 135, w4 86.7, 86.5;
//    464, K 256 w8 131, 128, w4 85, 79; 448, K 512 w8 132, 134;
//  * X units or more are left empty: 272 tiles, K 2048 w8 50.9, 55.9, w2 41.3, 42.7; 448, K 3584 w4 67, 74; 488, K 4096 w2 71, 80; 464 large ones, K 3072
//    w2 154, 168.
// With more rounds the sums of a round coincide: 768 large ones, 8192 x 6144, K 2048 269, 296; 1024, K 512 267, 258 to 265, 3584 478, 483 to 499.  (Consumers
// for all rounds but the last, own sums in that: 4096 x 8192, K 3584 258, 286; 8192 x 8192 473, 488.)
// Where the consumers sit in the grid decides when they run.  When the GEMM needs more than one
// chip-wide round of tiles, X consumers follow the first round of tiles: they take X compute
// units as the first tiles retire and keep them to the end, reducing finished tiles while the
// other units compute the next ones.  Behind the last tile sit as many consumers again as the
// chip has units; they pick up compute units as the last tiles retire and the whole chip
// finishes the queue.  All waits are bounded.  A consumer waits for flags of tiles that are ahead of it in the grid and of peers, a tile
// that sums for itself for peers' only, and emulated peers sit ahead of every tile.
//
// Sizing X: one work-group streams about 50 GB/s on its compute unit whatever it keeps in
// flight (measured; the whole chip reaches 5.4 TB/s only with all units streaming), so the
// reduction costs least unit-time when few units do it all along: X is the number of units
// that reduce the whole output in the time the remaining units need for the GEMM.
//
// The paper runs a persistent GEMM on a fixed set of compute units and the consumer as a second
// kernel on the rest, reducing through the switch (multimem).  Here there is no switch (the sum
// is done in software), and a persistent GEMM measured slower on this chip (its K loop ran 13 %
// slower than with one work-group per tile, which the dispatcher also load-balances).
#include "gemm_core.h"
#include "launch.h"
#include "reduce.h"

namespace ditron {

struct GemmArParams {
  const void* part[DITRON_MAX_WORLD];   // every rank's published partial [M, N] bf16; part[rank] is gemm_out
  const char* a;
  const char* b;
  __bf16* gemm_out;
  __bf16* out;
  int32_t* ticket;       // next position of the reduce queue
  int32_t* done;         // consumers that have left the queue
  int32_t* tile_flags;   // [world][ntiles]
  // two-shot only
  __bf16* out_dst[DITRON_MAX_WORLD];      // every rank's output buffer; out_dst[rank] is `out`
  const void* reduced[DITRON_MAX_WORLD];  // emulated peers: what rank s broadcasts (only the tiles it owns are read)
  int32_t* peer_done;                     // [world]: rank s has broadcast all its tiles
  int32_t* prod_count;                    // arrival counter of the emulated peers
  int32_t* status;
  int32_t* schedule;
  int m, n, k, world, rank;
  int32_t epoch;
  unsigned spin_limit;
  int num_producers;
  int head_tiles;        // tiles ahead of the early consumers
  int early, late;       // consumers behind the first round of tiles / behind the last tile
  int own_sums;          // a tile's work-group adds the peers' copies itself, there are no consumers (one-shot)
  int peers_resident;    // flags preset: the peers' partials are complete, only the own tile flags are waited for
  int group_m, num_xcd, per_xcd, npm, npn;
};

constexpr int kOwnSumColumns = 1 << 22;   // the most columns with which a tile's rows lie within 32-bit offsets

__device__ __forceinline__ void ar_tile_at(const GemmArParams& p, int position, int ntiles, int& pid_m, int& pid_n) {
  const int id = xcd_remap(position, ntiles, p.num_xcd, p.per_xcd);
  grouped_order(id, p.npm, p.npn, p.group_m, pid_m, pid_n);
}

// Sum of the `world` published copies of one output tile.  U vectors of 16 bytes per lane and
// rank are in flight at once (a single work-group owns its compute unit, so the loads in
// flight per lane are what fills the memory pipe).
template <class T, int WORLD, int U, bool TWO>
__device__ __forceinline__ void ar_reduce_tile(const GemmArParams& p, int m0, int n0) {
  const int world = WORLD > 0 ? WORLD : p.world;
  const int tile_m = min(T::BM, p.m - m0), tile_n = min(T::BN, p.n - n0);
  const int vpr = tile_n >> 3;                 // 16-byte vectors per tile row
  const int nvec = tile_m * vpr;
  const size_t ld = (size_t)p.n >> 3;          // vectors per matrix row
  const size_t base = (size_t)m0 * ld + ((size_t)n0 >> 3);
  u32x4_t* out = (u32x4_t*)p.out;
  for (int v0 = threadIdx.x; v0 < nvec; v0 += T::THREADS * U) {
    size_t off[U];
    u32x4_t x[U][WORLD > 0 ? WORLD : 1];
    float acc[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * T::THREADS;
      const int row = tile_n == T::BN ? v / (T::BN / 8) : v / vpr;
      const int col = v - row * vpr;
      off[u] = base + (size_t)row * ld + col;
      if (v < nvec) {
        if constexpr (WORLD > 0) {
#pragma unroll
          for (int s = 0; s < WORLD; ++s) x[u][s] = __builtin_nontemporal_load((const u32x4_t*)p.part[s] + off[u]);
        } else {
          set_bf16x8(acc[u], __builtin_nontemporal_load((const u32x4_t*)p.part[0] + off[u]));
          for (int s = 1; s < world; ++s) add_bf16x8(acc[u], __builtin_nontemporal_load((const u32x4_t*)p.part[s] + off[u]));
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * T::THREADS;
      if (v < nvec) {
        if constexpr (WORLD > 0) {
          set_bf16x8(acc[u], x[u][0]);
#pragma unroll
          for (int s = 1; s < WORLD; ++s) add_bf16x8(acc[u], x[u][s]);
        }
        const u32x4_t r = pack_bf16x8(acc[u]);
        if constexpr (TWO) {   // the broadcast: the reduced tile goes to every rank's output
          for (int d = 0; d < world; ++d) __builtin_nontemporal_store(r, (u32x4_t*)p.out_dst[d] + off[u]);
        } else {
          __builtin_nontemporal_store(r, out + off[u]);
        }
      }
    }
  }
}

// One-shot in a tile's own work-group: the parked tile (this rank's partial, rounded as the peers read it) plus the peers' partials
// of it, in rank order.  U vectors of 16 bytes per lane and peer are in flight; they are dealt over the rows and columns that exist.
template <class T, int WORLD, int U>
__device__ __forceinline__ void ar_sum_parked(const GemmArParams& p, int m0, int n0, const char* lds) {
  typedef ParkedTile<T> P;
  constexpr uint32_t kOut = 0xF0000000;   // end of every buffer: kOwnSumColumns keeps a tile's rows below it
  const int world = WORLD > 0 ? WORLD : p.world;
  const int tile_m = min(T::BM, p.m - m0), tile_n = min(T::BN, p.n - n0);
  const int vpr = tile_n >> 3;                 // 16-byte vectors per tile row
  const int nvec = tile_m * vpr;
  const size_t first = (size_t)m0 * p.n + n0;
  // (the own partial's buffer is empty: its loads cost nothing)
  auto rows_of = [&](int s) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const __bf16*)p.part[s] + first), 0, s == p.rank ? 0 : (int)kOut, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc((void*)(p.out + first), 0, (int)kOut, 0x00020000);
#pragma unroll 1
  for (int v0 = threadIdx.x; v0 < nvec; v0 += T::THREADS * U) {
    uint32_t off[U];
    const char* own[U];
    u32x4_t x[WORLD > 0 ? WORLD : 1][U];
    float acc[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * T::THREADS;
      const int row = tile_n == T::BN ? v / (T::BN / 8) : v / vpr;
      const int col = v - row * vpr;
      off[u] = v < nvec ? ((uint32_t)row * (uint32_t)p.n + (uint32_t)col * 8u) * 2u : kOut;
      // the wave that parked it, its row and slot there (a vector past the tile reads some parked one and is not stored)
      const int r = row % T::WTM, g = col % P::SL;
      own[u] = lds + ((row / T::WTM % T::WAVES_M * T::WAVES_N + col / P::SL) * T::WTM + r) * P::ROW + (g ^ P::key(r)) * 16;
    }
    if constexpr (WORLD > 0) {
#pragma unroll
      for (int s = 0; s < WORLD; ++s) {
        const __amdgpu_buffer_rsrc_t rows = rows_of(s);
#pragma unroll
        for (int u = 0; u < U; ++u) x[s][u] = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)off[u], 0, kStreaming);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const u32x4_t mine = *(const u32x4_t*)own[u];
        set_bf16x8(acc[u], p.rank == 0 ? mine : x[0][u]);
#pragma unroll
        for (int s = 1; s < WORLD; ++s) add_bf16x8(acc[u], s == p.rank ? mine : x[s][u]);
      }
    } else {
      for (int s = 0; s < world; ++s) {
        const __amdgpu_buffer_rsrc_t rows = rows_of(s);
#pragma unroll
        for (int u = 0; u < U; ++u) x[0][u] = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)off[u], 0, kStreaming);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const u32x4_t term = s == p.rank ? *(const u32x4_t*)own[u] : x[0][u];
          if (s == 0) set_bf16x8(acc[u], term);
          else add_bf16x8(acc[u], term);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) __builtin_amdgcn_raw_buffer_store_b128(pack_bf16x8(acc[u]), out, (int)off[u], 0, kStreaming);
  }
}

// Two-shot, emulated peers: one tile of what a peer broadcasts lands in the local output.
template <class T>
__device__ __forceinline__ void ar_copy_tile(const GemmArParams& p, const void* src, int m0, int n0) {
  const int tile_m = min(T::BM, p.m - m0), tile_n = min(T::BN, p.n - n0);
  const int vpr = tile_n >> 3;
  const int nvec = tile_m * vpr;
  const size_t ld = (size_t)p.n >> 3;
  const size_t base = (size_t)m0 * ld + ((size_t)n0 >> 3);
  constexpr int U = 8;
  for (int v0 = threadIdx.x; v0 < nvec; v0 += T::THREADS * U) {
    size_t off[U];
    u32x4_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * T::THREADS;
      const int row = v / vpr;
      off[u] = base + (size_t)row * ld + (v - row * vpr);
      if (v < nvec) x[u] = __builtin_nontemporal_load((const u32x4_t*)src + off[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v0 + u * T::THREADS < nvec) __builtin_nontemporal_store(x[u], (u32x4_t*)p.out + off[u]);
  }
}

// TWO: the two-shot form.  Position q of the tile order belongs to rank q % world; a rank reduces only
// its own tiles and stores each reduced tile into every rank's output; the other tiles of its output
// arrive from their owners.
template <class T, int WORLD, bool TWO>
__global__ __launch_bounds__(T::THREADS) void gemm_ar_kernel(const GemmArParams p) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int ntiles = p.npm * p.npn;
  int wg = blockIdx.x;
  if (wg < p.num_producers) {
    // emulated peers: flag (peer, tile) for every peer, tiles in schedule order
    const int peers = p.world - 1;
    const int total = peers * ntiles;
    for (int i = wg * T::THREADS + (int)threadIdx.x; i < total; i += p.num_producers * T::THREADS) {
      int s = i % peers;
      if (s >= p.rank) ++s;
      int pid_m, pid_n;
      ar_tile_at(p, i / peers, ntiles, pid_m, pid_n);
      flag_raise_stored(p.tile_flags + (size_t)s * ntiles + pid_m * p.npn + pid_n, p.epoch);   // (the partials were there before the launch)
    }
    if constexpr (TWO) {
      // the peers' broadcasts: the i-th tile that is not ours is position (i / (W-1)) W + s, s the
      // (i % (W-1))-th rank other than ours
      for (int i = wg;; i += p.num_producers) {
        const int block = (i / peers) * p.world;     // first position of the block of `world` positions
        if (block >= ntiles) break;
        int s = i % peers;
        if (s >= p.rank) ++s;
        const int q = block + s;
        if (q >= ntiles) continue;
        int pid_m, pid_n;
        ar_tile_at(p, q, ntiles, pid_m, pid_n);
        ar_copy_tile<T>(p, p.reduced[s], pid_m * T::BM, pid_n * T::BN);
      }
      // (no release: nothing of this launch reads the output, its end publishes it)
      stores_done();
      __syncthreads();
      if (threadIdx.x == 0) {
        const int old = __hip_atomic_fetch_add(p.prod_count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == p.num_producers - 1) {
          __hip_atomic_store(p.prod_count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          for (int r = 0; r < p.world; ++r)
            if (r != p.rank) flag_raise_stored(p.peer_done + r, p.epoch);
        }
      }
    }
    return;
  }
  wg -= p.num_producers;
  // grid: head_tiles tiles, `early` consumers, the remaining tiles, `late` consumers
  int pos = -1;
  if (wg < p.head_tiles) pos = wg;
  else if (wg >= p.head_tiles + p.early && wg < ntiles + p.early) pos = wg - p.early;

  if (pos >= 0) {
    int pid_m, pid_n;
    ar_tile_at(p, pos, ntiles, pid_m, pid_n);
    const int m0 = pid_m * T::BM, n0 = pid_n * T::BN;
    if (p.schedule && threadIdx.x == 0) {
      int32_t* rec = p.schedule + 4 * (size_t)pos;
      rec[0] = pid_m; rec[1] = pid_n; rec[2] = wg; rec[3] = 0;
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
    store_tile_bf16<T, true>(acc, p.gemm_out, (size_t)p.n, m0, n0, M, N, lds);
    // Summed here: every wave looks at the peers' flags once while its stores are on their way (it waits for them only after this
    // rank's own flag is up, so that ranks which wait for each other cannot block).
    const bool sums = !TWO && p.own_sums;
    const int lane = threadIdx.x & 63;
    const bool gate = sums && !p.peers_resident && lane < p.world && lane != p.rank;
    const int32_t* flag = p.tile_flags + (size_t)(gate ? lane : 0) * ntiles + pid_m * p.npn + pid_n;
    const bool up = !gate || __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == p.epoch;
    stores_done();
    __syncthreads();   // every wave's part of the tile is in memory: notify
    if (threadIdx.x == 0) flag_raise_stored(p.tile_flags + (size_t)p.rank * ntiles + pid_m * p.npn + pid_n, p.epoch);
    if constexpr (!TWO) {
      if (sums) {
        if (!up) flag_wait_lane(p.tile_flags + (size_t)lane * ntiles, pid_m * p.npn + pid_n, 1, p.epoch, p.spin_limit, p.status);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const int nvec = min(T::BM, p.m - m0) * (min(T::BN, p.n - n0) >> 3);
        if (nvec <= 2 * T::THREADS) ar_sum_parked<T, WORLD, 2>(p, m0, n0, lds);
        else if (T::BM == 256 || nvec <= 4 * T::THREADS) ar_sum_parked<T, WORLD, 4>(p, m0, n0, lds);
        else ar_sum_parked<T, WORLD, 8>(p, m0, n0, lds);
      }
    }
    return;
  }

  // a consumer: draw tickets until the queue is empty
  volatile int* drawn = (volatile int*)lds;
  for (;;) {
    __syncthreads();   // the previous ticket has been read by every wave
    if (threadIdx.x == 0) *drawn = __hip_atomic_fetch_add(p.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int q = TWO ? *drawn * p.world + p.rank : *drawn;   // two-shot: only the positions this rank owns
    if (q >= ntiles) break;
    int pid_m, pid_n;
    ar_tile_at(p, q, ntiles, pid_m, pid_n);
    if ((int)threadIdx.x < p.world && (!p.peers_resident || (int)threadIdx.x == p.rank))
      flag_wait_lane(p.tile_flags + (size_t)threadIdx.x * ntiles, pid_m * p.npn + pid_n, 1, p.epoch, p.spin_limit, p.status);
    __syncthreads();
    ar_reduce_tile<T, WORLD, WORLD == 2 || WORLD == 4 ? 8 : 4, TWO>(p, pid_m * T::BM, pid_n * T::BN);
  }
  // the last consumer to leave puts the queue back to zero for the next call
  if (threadIdx.x == 0) {
    // (relaxed: the count guards nothing but the two words below, and every consumer's last ticket has been drawn before it counts itself)
    const int old = __hip_atomic_fetch_add(p.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == p.early + p.late - 1) {
      if constexpr (TWO) {
        // the output is complete when the call returns: the peers' broadcasts must have landed too
        for (int r = 0; r < p.world; ++r)
          if (r != p.rank) flag_wait_lane(p.peer_done, r, 1, p.epoch, p.spin_limit, p.status);
      }
      __hip_atomic_store(p.ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(p.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

template <auto Kernel>
struct KernelConstant {
  static constexpr auto value = Kernel;
};

template <class T>
static ditron_status_t launch_ar(GemmArParams& p, int units, bool two_shot, hipStream_t stream) {
  const int ntiles = p.npm * p.npn;
  units = units / 8 * 8;
  p.head_tiles = std::min(ntiles, units);
  // X units reduce while units - X compute the tiles at the per-unit MFMA rate of a full-chip GEMM:
  // balance the two.  Per GEMM tile the consumer moves (world + 1) tile-sized streams in the one-shot
  // form and 2 in the two-shot form (world reads and world writes for one tile in `world`), at ~40 GB/s
  // per unit (50 while streaming, less the waits).
  constexpr double kUnitBytes = 40e9, kUnitFlops = 5.3e12;   // (measured at table shape 3: X = 40 / 56 / 64 / 72 / 80 -> 555 / 534 / 528 / 540 / 545 us)
  const double streams = two_shot ? 2.0 : p.world + 1.0;
  const double t_reduce = streams * T::BM * T::BN * 2 / kUnitBytes;   // unit-seconds per tile
  const double t_gemm = 2.0 * T::BM * T::BN * p.k / kUnitFlops;
  const int x = std::min((int)(units * t_reduce / (t_reduce + t_gemm) / 8 + 0.5) * 8, units / 2);
  // One round of tiles: the tiles sum.  Two rounds that leave fewer than X units empty: the X consumers would push a part of the tiles into a
  // third round, which costs about a t_gemm; the tiles' own sums coincide in both rounds instead, which costs more the shorter the
  // contraction is against the number of ranks (figures of both sides at the top of the file).  So the tiles sum if t_gemm is three
  // times t_reduce or more (256-row tiles: three and a half); and, 256-row tiles, if it is half of it or less: memory is then the bound, and
  // a tile's sum reads one copy less of it.
  const bool third_round = ntiles > 2 * units - x && ntiles <= 2 * units;
  const bool memory_bound = T::BM == 256 && t_reduce >= 2 * t_gemm && ntiles > 2 * units - units / 4;
  p.own_sums = !two_shot && p.n <= kOwnSumColumns && (ntiles <= units || (third_round && (t_gemm >= (T::BM == 256 ? 3.5 : 3.0) * t_reduce || memory_bound)));
  p.early = !p.own_sums && ntiles > units ? x : 0;
  p.late = p.own_sums ? 0 : std::min(units, ntiles);
  const unsigned grid = (unsigned)(p.num_producers + ntiles + p.early + p.late);
  auto launch = [&](auto instance) {
    constexpr auto kern = decltype(instance)::value;
    if (!set_dynamic_lds<kern>(T::LDS_BYTES)) return DITRON_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(T::THREADS), T::LDS_BYTES, stream, p);
    return hipGetLastError() == hipSuccess ? DITRON_OK : DITRON_ERR_HIP;
  };
  // a fixed number of ranks lets the consumer have the vectors of every rank in flight together
  switch (p.world) {
    case 2: return two_shot ? launch(KernelConstant<gemm_ar_kernel<T, 2, true>>{}) : launch(KernelConstant<gemm_ar_kernel<T, 2, false>>{});
    case 4: return two_shot ? launch(KernelConstant<gemm_ar_kernel<T, 4, true>>{}) : launch(KernelConstant<gemm_ar_kernel<T, 4, false>>{});
    case 8: return two_shot ? launch(KernelConstant<gemm_ar_kernel<T, 8, true>>{}) : launch(KernelConstant<gemm_ar_kernel<T, 8, false>>{});
    default: return two_shot ? launch(KernelConstant<gemm_ar_kernel<T, 0, true>>{}) : launch(KernelConstant<gemm_ar_kernel<T, 0, false>>{});
  }
}

}  // namespace ditron

using namespace ditron;

static ditron_status_t gemm_ar_impl(const void* a, const void* b, int b_layout, void* gemm_out,
                                    const void* const* peer_partials, void* out, void* const* out_dsts,
                                    const void* const* peer_reduced, int32_t* signals, int32_t* status,
                                    int32_t* schedule_out, int m, int n, int k_local, int world, int rank,
                                    int32_t epoch, unsigned flags, const ditron_tuning_t* tuning, void* stream) {
  const bool two_shot = out_dsts != nullptr;

  if (world < 1 || world > DITRON_MAX_WORLD || rank < 0 || rank >= world) return DITRON_ERR_INVALID_ARG;
  if (m <= 0 || n <= 0 || k_local <= 0) return DITRON_ERR_INVALID_ARG;
  if (!a || !b || !gemm_out || !out || !signals || !status || out == gemm_out) return DITRON_ERR_INVALID_ARG;
  if (world > 1 && !peer_partials) return DITRON_ERR_INVALID_ARG;
  if (!aligned16(a) || !aligned16(b) || !aligned16(gemm_out) || !aligned16(out) || !aligned16(signals))
    return DITRON_ERR_INVALID_ARG;
  const Mode mode = producer_mode(flags);
  if (flags & DITRON_EPOCH_IN_MEMORY) return DITRON_ERR_UNSUPPORTED;
  const Tuning tune = resolve_tuning(tuning, 1);
  if (mode == Mode::kInvalid || !tune.valid) return DITRON_ERR_INVALID_ARG;
  if (mode == Mode::kPreset && two_shot) return DITRON_ERR_UNSUPPORTED;   // the peers' broadcasts are part of the call
  const bool emulate = mode == Mode::kEmulate;
  if ((flags & DITRON_DUMP_SCHEDULE) && !schedule_out) return DITRON_ERR_INVALID_ARG;
  if (b_layout != DITRON_B_KN && b_layout != DITRON_B_NK) return DITRON_ERR_INVALID_ARG;
  if (k_local % 8 != 0 || n % 8 != 0) return DITRON_ERR_UNSUPPORTED;
  if (!fits_32bit(m, k_local, 2) || !fits_32bit(n, k_local, 2)) return DITRON_ERR_UNSUPPORTED;

  GemmArParams p{};
  if (two_shot) {
    for (int s = 0; s < world; ++s) {
      if (!out_dsts[s] || !aligned16(out_dsts[s]) || out_dsts[s] == gemm_out) return DITRON_ERR_INVALID_ARG;
      p.out_dst[s] = (__bf16*)out_dsts[s];
      if (s != rank && emulate) {
        if (!peer_reduced || !peer_reduced[s] || !aligned16(peer_reduced[s]) || peer_reduced[s] == out)
          return DITRON_ERR_INVALID_ARG;
        p.reduced[s] = peer_reduced[s];
      }
    }
  }
  for (int s = 0; s < world; ++s) {
    if (s == rank) {
      p.part[s] = gemm_out;
    } else {
      if (!peer_partials[s] || !aligned16(peer_partials[s]) || peer_partials[s] == out) return DITRON_ERR_INVALID_ARG;
      p.part[s] = peer_partials[s];
    }
  }
  const TileChoice tc = choose_tile(m, n, k_local, Narrow::kAllReduce);
  p.npm = cdiv(m, tc.block_m);
  p.npn = cdiv(n, tc.block_n);
  const int ntiles = p.npm * p.npn;
  int dev = 0, units = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || units < 16)
    return DITRON_ERR_HIP;
  p.a = (const char*)a;
  p.ticket = signals;
  p.done = signals + 1;
  p.b = (const char*)b;
  p.gemm_out = (__bf16*)gemm_out;
  p.out = (__bf16*)out;
  p.tile_flags = signals + 2 * world;
  p.peer_done = signals + 2 * world + (size_t)world * ntiles;
  p.prod_count = signals + 2;
  p.status = status;
  p.schedule = (flags & DITRON_DUMP_SCHEDULE) ? schedule_out : nullptr;
  p.m = m;
  p.n = n;
  p.k = k_local;
  p.world = world;
  p.rank = rank;
  p.epoch = epoch;
  p.spin_limit = tune.spin_limit;
  p.peers_resident = mode == Mode::kPreset;
  // one-shot: the emulated peers only raise flags; two-shot: they also copy the peers' broadcasts
  p.num_producers = (emulate && world > 1) ? (two_shot ? 64 : 8) : 0;
  p.group_m = tc.group_m;
  p.num_xcd = tc.num_xcd;
  p.per_xcd = tc.per_xcd;
  const hipStream_t s = (hipStream_t)stream;
  const bool kn = b_layout == DITRON_B_KN;
  if (!tc.big) return kn ? launch_ar<TileSmallKN>(p, units, two_shot, s) : launch_ar<TileSmall>(p, units, two_shot, s);
  return kn ? launch_ar<TileBigKN>(p, units, two_shot, s) : launch_ar<TileBigDirect>(p, units, two_shot, s);
}

extern "C" ditron_status_t ditron_gemm_ar(const void* a, const void* b, int b_layout, void* gemm_out,
                                          const void* const* peer_partials, void* out, int32_t* signals,
                                          int32_t* status, int32_t* schedule_out, int m, int n, int k_local,
                                          int world, int rank, int32_t epoch, unsigned flags,
                                          const ditron_tuning_t* tuning, void* stream) {
  return gemm_ar_impl(a, b, b_layout, gemm_out, peer_partials, out, nullptr, nullptr, signals, status, schedule_out, m, n,
                      k_local, world, rank, epoch, flags, tuning, stream);
}

extern "C" ditron_status_t ditron_gemm_ar_two_shot(const void* a, const void* b, int b_layout, void* gemm_out,
                                                   const void* const* peer_partials, void* const* out_dsts,
                                                   const void* const* peer_reduced, int32_t* signals,
                                                   int32_t* status, int32_t* schedule_out, int m, int n,
                                                   int k_local, int world, int rank, int32_t epoch, unsigned flags,
                                                   const ditron_tuning_t* tuning, void* stream) {
  if (!out_dsts || world < 1 || world > DITRON_MAX_WORLD || rank < 0 || rank >= world) return DITRON_ERR_INVALID_ARG;
  return gemm_ar_impl(a, b, b_layout, gemm_out, peer_partials, out_dsts[rank], out_dsts, peer_reduced, signals, status,
                      schedule_out, m, n, k_local, world, rank, epoch, flags, tuning, stream);
}
