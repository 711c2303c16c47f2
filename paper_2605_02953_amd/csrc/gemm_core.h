// MFMA tile engine for gfx950, bf16 and OCP e4m3: C_tile[BM,BN] (fp32) += A_tile[BM,K] . B_tile[BN,K]^T.
//
// Both operands are read as rows that are contiguous along the contraction dimension (bf16: B also stored [K, N], see B_KN).  A
// K slice of 128 bytes of BM + BN rows is staged in LDS as 128-byte rows (one cache line per
// row) whose eight 16-byte chunks are XOR-swizzled by the row index.  Four waves, one per SIMD,
// each own a quarter of the tile and feed v_mfma_f32_16x16x32_bf16, v_mfma_f32_16x16x128_f8f6f4 or, for a few MoE tiles,
// v_mfma_f32_32x32x16_bf16 from 128-bit LDS reads.  The
// instruction's row operand is taken from the B rows and its column operand from the A rows,
// so that a lane ends up with four consecutive output columns of one output row.
#pragma once
#include <type_traits>
#include "common.h"

namespace ditron {

// 16 zero bytes in global memory, for kernels that stage operands with the direct-to-LDS load
// (it has no per-lane zero fill): lanes whose K-chunk lies beyond the contraction length stage
// these instead.
__device__ const u32x4_t kZeroChunk = {0u, 0u, 0u, 0u};

// Chunk swizzle for 128-byte LDS rows (eight 16-byte chunks): chunk c of row r is stored at
// chunk position c ^ swz128(r).  Makes 128-bit reads of 8 or of 16 consecutive rows at one
// logical chunk hit distinct banks; invariant under adding a multiple of 16 rows.
__device__ __forceinline__ int swz128(int r) { return (r & 7) ^ ((r >> 3) & 1); }
// The same for the 16 x 16 x 32 form, whose 128-bit reads take the four chunks of a 32-deep step of 16
// consecutive rows (lane = 16 chunk + row): measured on the chip with the LDS saturated, that read takes 1.64
// times as long under swz128 as under this one (and the 32-row read above 1.64 times as long under this one).
__device__ __forceinline__ int swz128_x16(int r) { return r & 7; }

// The same for a B tile staged as k rows of BN elements: the pair of 16-byte chunks p (16 columns) of k row r is stored at
// pair position p ^ swz_kn<BN>(r).  A transposing read takes four rows (r .. r + 3, r a multiple of 4) of one pair per group
// of 16 lanes, two groups (rows 8 apart) per cycle: eight pairs that fall on the eight 32-byte windows of the 256-byte bank
// row.  Rows of 256 and 128 elements all start at window 0; rows of 192 at window 4 r mod 8 (and the exclusive or stays below
// their 12 pairs); rows of 224 at window 6 r mod 8, where flipping bit 0 for the rows 8 apart is enough (14 pairs);
// rows of 64 at window 4 r mod 8, so bit 0 tells the rows 2 apart from each other and bit 1 those 8 apart (four pairs).
template <int BN>
__device__ __forceinline__ int swz_kn(int r) {
  static_assert(BN == 256 || BN == 224 || BN == 192 || BN == 128 || BN == 64, "bank windows worked out for these");
  if (BN == 64) return ((r >> 1) & 1) | ((r >> 2) & 2);
  if (BN == 224) return (r >> 3) & 1;
  return BN == 192 ? (r & 2) | ((r >> 3) & 1) : (r & 3) | ((r >> 1) & 4);
}

// The explicit waits are pinned in place: the scheduler must not move matrix instructions
// behind them (a wave blocked in a wait issues nothing).
__device__ __forceinline__ void wait_vmcnt0() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __builtin_amdgcn_sched_barrier(0);
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt immediate (six bits: [3:0] and [15:14])");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void wait_lgkmcnt0() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_sched_barrier(0);
}

// Work-group barrier that leaves outstanding global loads in flight (the plain
// __syncthreads() drains them).  The empty asm statements stop the compiler from moving
// memory accesses across it; sched_barrier keeps the instruction scheduler from moving
// anything else (the phases of the two wave groups must not be blended).
__device__ __forceinline__ void barrier_no_drain() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// ------------------------------------------------------------------ the tile
// BM x BN output tile (BM 256 or 128, BN 256, 224, 192, 128 or 64) computed by four waves, one per SIMD,
// each owning BM/2 x BN/2 (256 x 256: 128 x 128 per wave, 256 accumulator registers, every
// fragment read from LDS feeds four MFMAs).
//
// X16: operands go global -> LDS (DIRECT: `buffer_load ... lds`) into a ring of operand pieces and feed
// v_mfma_f32_16x16x32_bf16 (a wave's quarter is cut into 16 x 16 blocks, a fragment is 16 rows x 32 k: the 16-byte chunk
// (lane / 16) of the 32-deep step of row (lane % 16)).  The accumulator of a block is four registers instead of sixteen, so
// the instruction moves a quarter of the accumulator registers per unit of matrix work.  LDS rows of 128 bytes (measured
// free of bank conflicts for the fragment reads).
// Otherwise: operands go global -> registers -> LDS (or, DIRECT, through gemm_mainloop_ring_split) in two stages of one
// 64-deep K tile each and feed v_mfma_f32_32x32x16_bf16: the MoE tiles for which that measured faster.
//
// B_KN (X16): B is stored [K, N] (N contiguous) instead of [N, K].  Its K tile is staged as it lies in memory, 64 rows of
// BN elements, the pairs of chunks swizzled by the row (swz_kn), and the MFMA operand (eight consecutive k of one column per
// lane) is assembled by two transposing LDS reads (ds_read_b64_tr_b16: inside each group of 16 lanes, lane i receives
// element i % 4 of the 8-byte chunks addressed by lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4; measured).  Everything that counts
// in bytes is as for [N, K].  (It replaced a register-staged 32 x 32 x 16 loop: [7976 x 8192] x [8192 x 3584] fused 441 ->
// 394 us at 256 x 256 tiles, 128 x 128 tiles 20 to 30 % less, MoE, with the blocks that it then takes, 0 to 25 % less.)
//
// F8: both operands are OCP e4m3 (a 128-byte row of a K tile is 128 elements), fed to v_mfma_f32_16x16x128_f8f6f4 by a
// loop of its own (gemm_mainloop_f8); everything that counts in bytes is as for X16.  `K` is then passed in units of
// two bytes.
//
// DEPTH_: K tiles requested ahead by the X16 loop, 0 = as many as the tile does best with on its own unit.
template <int BM_, int BN_, bool B_KN_ = false, bool DIRECT_ = false, bool X16_ = false, bool F8_ = false, int DEPTH_ = 0>
struct GemmTile4W {
  static_assert((BM_ == 256 || BM_ == 128) && (BN_ == 256 || BN_ == 192 || BN_ == 128 || (X16_ && BN_ == 224) || (X16_ && BM_ == 128 && BN_ == 64)), "supported tile sides");
  static_assert(!B_KN_ || X16_, "the 32 x 32 x 16 loop is written for [N, K] operands");
  static_assert(!X16_ || DIRECT_, "the 16 x 16 x 32 loop is written for the direct-to-LDS staging");
  static_assert(!F8_ || (X16_ && !B_KN_ && BM_ == 256 && BN_ >= 192), "the fp8 loop is written for 256-row tiles and direct-to-LDS staging");
  static_assert(!X16_ || BN_ % 32 == 0, "whole 16 x 16 blocks per wave");
  static constexpr bool B_KN = B_KN_;
  static constexpr bool DIRECT = DIRECT_;   // operands go from global memory straight into LDS (no staging registers)
  static constexpr bool X16 = X16_;
  static constexpr bool F8 = F8_;
  static constexpr int BM = BM_, BN = BN_, BK = 64, NSTAGE = 2;
  static constexpr int WAVES_M = 2, WAVES_N = 2, NWAVES = 4, THREADS = 256;
  static constexpr int WTM = BM / 2, WTN = BN / 2, MI = WTM / 32, NI = WTN / 32;
  static constexpr int ROW_BYTES = 128;
  static constexpr int PB = BN * 2;                           // B_KN: bytes of a k row of the staged B tile
  static constexpr int A_BYTES = BM * ROW_BYTES, B_BYTES = BN * ROW_BYTES;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  // X16: a ring of 2 DEPTH + 1 operand pieces (the A part and the B part of a K tile are pieces of their own): DEPTH K
  // tiles are requested ahead.  256 rows: five pieces are all of the LDS.  128 rows: seven of ten (2 / 3 / 4 tiles ahead,
  // [1024 x 8192] x [8192 x 3696], operands resident: 66 / 57 / 57 us; 464 tiles of [2048 x 3696]: 123 / 109 / 111 us, so a
  // second work-group on the unit, which 2 would leave room for, is worth less than the third tile in flight).  64 columns:
  // nine, their calls stream the weight from memory.
  // B parts larger than A parts (128 rows, 192 or 256 columns): a ring of DEPTH + 1 A parts and behind it one of DEPTH B parts,
  // since in pieces of one size half of the A parts' room would be empty and two K tiles all that fits (MoE, [k, n] weights not in
  // the caches, whole calls: 60 experts, 4856 tokens top-2, hidden 4096, 512 columns 125 -> 112 us; 16 experts, 5064 tokens,
  // hidden 2048, 1024 columns 76 -> 70; 42 calls more of K 1024 to 4096: 2 to 16 % less).  The 256-row tiles lose 1 to 2 % with two
  // rings.
  static constexpr bool TWO_RINGS = X16_ && B_BYTES > A_BYTES;
  static constexpr int PIECE_BYTES = A_BYTES;
  static constexpr int DEPTH = DEPTH_ ? DEPTH_ : BN == 64 ? 4 : BM == 128 ? 3 : 2;
  static constexpr int PIECES = 2 * DEPTH + 1;
  static constexpr int LDS_BYTES = TWO_RINGS ? (DEPTH + 1) * A_BYTES + DEPTH * B_BYTES : X16_ ? PIECES * PIECE_BYTES : NSTAGE * STAGE_BYTES;
  static constexpr int ROWS_PER_PASS = THREADS / 8;           // 32 rows per pass of 16-byte loads
  static constexpr int A_LOADS = BM / ROWS_PER_PASS, B_LOADS = BN / ROWS_PER_PASS, LOADS = A_LOADS + B_LOADS;
  // The K loop is written as slots of two MFMAs (one B fragment, two A fragments).
  static constexpr int PAIRS = MI * NI / 2;                   // slots per 16-deep step
  static constexpr int SLOTS = 4 * PAIRS;                     // slots per 64-deep K tile
  static constexpr int B_READS = B_KN ? 2 : 1;                // X16: LDS reads per B fragment
  static constexpr int READS = MI + NI;                       // fragment reads per step (32 x 32 x 16 loop)
  static constexpr int HALF = (PAIRS + 1) / 2;                // slots of a step that take its reads when they must be early
  static constexpr int MB = WTM / 16, NB = WTN / 16;          // X16: 16 x 16 blocks of a wave's quarter
  // the accumulators of one wave: [column block][row block]
  typedef f32x16_t Acc32[NI][MI];
  typedef f32x4_t Acc16[NB][MB];
  typedef std::conditional_t<X16_, Acc16, Acc32> Acc;
};

template <class T>
struct Frags4W {
  bf16x8_t a[T::MI], b[T::NI];
};

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

typedef short s16x4_t __attribute__((ext_vector_type(4)));

// Fragment read J of step KS (0..3) of the K tile staged at `st`.  koff[KS] is the lane's
// swizzled chunk offset for that step.  The order (b0, a0..a[MI-1], b1..b[NI-1]) is the order
// in which mma_pair consumes them.
template <class T, int KS, int J>
__device__ __forceinline__ void read_one(Frags4W<T>& f, const char* st, int a_off, int b_off, const int (&koff)[4]) {
  if constexpr (J == 0) f.b[0] = *(const bf16x8_t*)(st + b_off + koff[KS]);
  else if constexpr (J <= T::MI) f.a[J - 1] = *(const bf16x8_t*)(st + a_off + (J - 1) * 32 * 128 + koff[KS]);
  else f.b[J - T::MI] = *(const bf16x8_t*)(st + b_off + (J - T::MI) * 32 * 128 + koff[KS]);
}
// reads [LO, HI) of a step
template <class T, int KS, int LO, int HI>
__device__ __forceinline__ void read_range(Frags4W<T>& f, const char* st, int a_off, int b_off, const int (&koff)[4]) {
  static_for<LO, HI>([&](auto j) { read_one<T, KS, decltype(j)::value>(f, st, a_off, b_off, koff); });
}

template <class T, int P>
__device__ __forceinline__ void mma_pair(typename T::Acc32& acc, const Frags4W<T>& f) {
  constexpr int ni = P / (T::MI / 2), mi = (P % (T::MI / 2)) * 2;
  acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[ni], f.a[mi], acc[ni][mi], 0, 0, 0);
  acc[ni][mi + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[ni], f.a[mi + 1], acc[ni][mi + 1], 0, 0, 0);
}

// Where the columns of a B stored [K, N] are: the mainloop's `b_row` argument for B_KN tiles.
struct BColumns {
  uint32_t ld_bytes;   // bytes between two k rows (2 N)
  int n0, n;           // first column of the tile, number of columns of B
};

template <class T>
struct Stager4W {
  static constexpr int kOutOfRange = 0x7ffffff0;
  static constexpr int KN_LANES = T::BN / 8;              // B_KN: lanes that cover one k row of the tile
    static constexpr bool kDirect = T::DIRECT;
  __amdgpu_buffer_rsrc_t a_rsrc, b_rsrc;
  int off[T::LOADS];
  u32x4_t reg[T::LOADS];
  int lds_off;    // byte offset inside an operand area of a stage, pass 0
  int kc;
  int kn_tid, kn_tile_bytes;   // B_KN: the lane's place among the loading threads, bytes per K tile of B
  int wave_lds;   // direct-to-LDS form: where the wave's 8 rows of a pass start

  // B_KN: the k row that the lane's load of pass `pass` belongs to
  __device__ __forceinline__ int kn_row(int pass) const { return (pass * T::THREADS + kn_tid) / KN_LANES; }

  template <class ARow, class BRow>
  __device__ __forceinline__ void init(const char* a_base, ARow a_row, const char* b_base, BRow b_row) {
    init(a_base, a_row, b_base, b_row, (int)threadIdx.x);
  }
  // tid: the thread's index among the T::THREADS threads that stage (the whole work-group, or its loading waves)
  template <class ARow, class BRow>
  __device__ __forceinline__ void init(const char* a_base, ARow a_row, const char* b_base, BRow b_row, int tid) {
    const int r = tid >> 3;
    // direct-to-LDS form: the lane's LDS position is chunk (lane & 7) of its row, which holds global chunk c
    const int c = kDirect ? ((tid & 7) ^ (T::X16 ? swz128_x16(r) : swz128(r))) : (tid & 7);
    wave_lds = __builtin_amdgcn_readfirstlane(tid >> 6) * 1024;
    a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a_base, 0, kOutOfRange, 0x00020000);
    b_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)b_base, 0, kOutOfRange, 0x00020000);
    kc = c * 8;
    lds_off = r * T::ROW_BYTES + ((c ^ swz128(r)) * 16);
#pragma unroll
    for (int i = 0; i < T::A_LOADS; ++i) off[i] = (int)(a_row(r + i * T::ROWS_PER_PASS) + (uint32_t)(c * 16));
    if constexpr (T::B_KN) {
      // the staged rows follow each other without gaps: pass i and thread tid fill 16-byte chunk i THREADS + tid of them
      kn_tid = tid;
      kn_tile_bytes = (int)(b_row.ld_bytes * 64u);
#pragma unroll
      for (int i = 0; i < T::B_LOADS; ++i) {
        const int row = kn_row(i), n8 = i * T::THREADS + tid - row * KN_LANES;
        const int col = b_row.n0 + (n8 ^ (2 * swz_kn<T::BN>(row))) * 8;   // position n8 holds global chunk n8 ^ 2 swz_kn
        off[T::A_LOADS + i] = col < b_row.n ? (int)((uint32_t)row * b_row.ld_bytes + (uint32_t)col * 2u)
                                            : kOutOfRange;   // columns past N read as zero
      }
    } else {
#pragma unroll
      for (int i = 0; i < T::B_LOADS; ++i)
        off[T::A_LOADS + i] = (int)(b_row(r + i * T::ROWS_PER_PASS) + (uint32_t)(c * 16));
    }
  }

  // `kt` must be a valid K tile; a chunk past K reads as zero (lane offset pushed out of range)
  template <int I>
  __device__ __forceinline__ u32x4_t load_one(int kt, int K) const {
    const bool dead = kt * 64 + kc >= K;
    const int v = dead ? kOutOfRange : off[I];
    return __builtin_amdgcn_raw_buffer_load_b128(I < T::A_LOADS ? a_rsrc : b_rsrc, v, kt * 128, 0);
  }
  // Direct-to-LDS form of load I (B stored [K, N]: below; else): the wave's 64 lanes fill 8 rows x 128 bytes that are
  // contiguous in the stage (lane l lands at byte 16 l), so the swizzle is applied on the global side: `off`
  // was built for the chunk that belongs at the lane's LDS position.  A chunk past K is pushed out of the
  // buffer's range, for which zeros are written.  B stored [K, N]: the 64 lanes fill 1 KiB of k rows of BN elements.
  template <int I, bool WHOLE = false>
  __device__ __forceinline__ void issue_one(int kt, int K, char* stage) const {
    constexpr int area = I < T::A_LOADS ? 0 : T::A_BYTES;
    constexpr int pass = I < T::A_LOADS ? I : I - T::A_LOADS;
    constexpr bool kn = T::B_KN && I >= T::A_LOADS;   // rows of k, not chunks of k
    const bool dead = !WHOLE && kt * 64 + (kn ? kn_row(pass) : kc) >= K;   // WHOLE: K is a whole number of K tiles, nothing lies past it
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass does not know this builtin
    __builtin_amdgcn_raw_ptr_buffer_load_lds(I < T::A_LOADS ? a_rsrc : b_rsrc,
                                             DITRON_LDS(stage + area + pass * T::ROWS_PER_PASS * T::ROW_BYTES + wave_lds), 16,
                                             dead ? kOutOfRange : off[I], kt * (kn ? kn_tile_bytes : 128), 0, 0);
#else
    (void)dead; (void)stage;
#endif
  }
  template <int LO, int HI>
  __device__ __forceinline__ void issue_range(int kt, int K, char* stage) const {
    static_for<LO, HI>([&](auto i) { issue_one<decltype(i)::value>(kt, K, stage); });
  }
  template <int I>
  __device__ __forceinline__ void fetch_one(int kt, int K) { reg[I] = load_one<I>(kt, K); }
  template <int LO, int HI>
  __device__ __forceinline__ void fetch_range(int kt, int K) {
    static_for<LO, HI>([&](auto i) { fetch_one<decltype(i)::value>(kt, K); });
  }

  // `stage`: the stage that receives the K tile
  template <int I>
  __device__ __forceinline__ void commit_one(char* stage) const {
    constexpr int area = I < T::A_LOADS ? 0 : T::A_BYTES;
    constexpr int pass = I < T::A_LOADS ? I : I - T::A_LOADS;
    *(u32x4_t*)(stage + area + lds_off + pass * T::ROWS_PER_PASS * T::ROW_BYTES) = reg[I];
  }
  template <int LO, int HI>
  __device__ __forceinline__ void commit_range(char* stage) const {
    static_for<LO, HI>([&](auto i) { commit_one<decltype(i)::value>(stage); });
  }
};

// The K tile that a work-group of this chiplet begins with where rows are a multiple of 16 KiB apart (rows_share_channels): an eighth of
// the contraction after the chiplet before it.  A K tile takes 128 bytes of every row; at such distances the same 128 bytes of all rows
// share few memory channels, and work-groups that walk the contraction in step ask those few all at once.  Inside a chiplet they
// stay in step and share its L2.  (The order in which products are added changes with it, not their number or their format.)  128-row
// tiles of [n, k] operands, us with one beginning and with eight: AllGather-GEMM 1024 x 2560, K 16384 152 to 155, 135; 1024 x 3696, K 8192 72
// to 84, by card and by where the buffers fall, and 71 to 75; rows 8 KiB or less apart, K 4096, 512 x 6656 36.6, 36.8, 1024 x 3696 41.8, 42.1;
// [k, n] operands 64 x 3584, K 8192 40.0, 40.9; 256-row tiles, 8192 x 3584, 365, 367.  A beginning per column block instead of per chiplet
// costs the L2's sharing: 1024 x 3696 80 -> 81, 8192 x 3584 365 -> 395.  MoE, hidden 8192: 1024 tokens, 32 experts, 512 columns 102, 97;
// 4096 tokens top-2, 8 of 64 experts, 768 columns 112, 111; 256 tokens top-2, 8 experts, 1024 columns 85, 82.
__device__ __forceinline__ int chiplet_k_tile(int K) {
  return (int)((unsigned)(K / 64) * (blockIdx.x & 7u) >> 3);
}
__host__ __device__ inline bool rows_share_channels(int K) { return K % 8192 == 0; }

// ------------------------------------------------------------------ 16 x 16 x 32 form
// The transposing read beside direct-to-LDS loads.  A bare builtin call carries no alias information, and the compiler then
// waits for every load in flight (vmcnt(0)) before it, as if it might read what they write: the loop below took three times
// as long.  The restrict-qualified parameter gives it some; which loads have landed is the loop's own affair, as it is for
// the ordinary reads.
__device__ __forceinline__ bf16x4_t read_tr16(__attribute__((address_space(3))) s16x4_t* __restrict__ src) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_bit_cast(bf16x4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(src));
#else
  return bf16x4_t{};
#endif
}

template <class T>
struct Frags16 {
  bf16x8_t a[T::MB];
  bf16x4_t b[T::NB][2];   // low and high four k of the fragment ([N, K] storage fills both with one read)
};

// Fragment read J of the 32-deep step KS (0 or 1) of the K tile whose A part is staged at `pa` and whose B part
// at `pb`, in the order the slots below consume them: b0, a0 .. a[MB-1], b1 .. b[NB-1] (B stored [K, N]: two reads
// per B fragment).  koff[KS]: the lane's swizzled chunk offset; b_off: the row of its column or, B stored [K, N], per
// column block the 8 bytes it addresses in the transposing read.
template <class T, int KS, int J>
__device__ __forceinline__ void read_one16(Frags16<T>& f, const char* pa, const char* pb, int a_off, const int* b_off,
                                            const int (&koff)[2]) {
  constexpr int BR = T::B_READS;
  if constexpr (J >= BR && J < BR + T::MB) {
    f.a[J - BR] = *(const bf16x8_t*)(pa + a_off + (J - BR) * 16 * 128 + koff[KS]);
  } else {
    constexpr int JB = J < BR ? J : J - T::MB, NB_ = JB / BR;
    if constexpr (T::B_KN) {
      const char* src = pb + b_off[NB_] + (KS * 32 + (JB % BR) * 4) * T::PB;
      f.b[NB_][JB % BR] = read_tr16((__attribute__((address_space(3))) s16x4_t*)DITRON_LDS(src));
    } else {
      const bf16x8_t v = *(const bf16x8_t*)(pb + b_off[0] + NB_ * 16 * 128 + koff[KS]);
      f.b[NB_][0] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
      f.b[NB_][1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
    }
  }
}

// MFMA I (0..3) of slot S of a step: column block S / (MB / 4), row block 4 (S % (MB / 4)) + I.
template <class T, int S, int I>
__device__ __forceinline__ void mma_one16(typename T::Acc16& acc, const Frags16<T>& f) {
  constexpr int nb = S / (T::MB / 4), mb = (S % (T::MB / 4)) * 4 + I;
  const bf16x8_t b = __builtin_shufflevector(f.b[nb][0], f.b[nb][1], 0, 1, 2, 3, 4, 5, 6, 7);
  acc[nb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, f.a[mb], acc[nb][mb], 0, 0, 0);
}

// The N loads of a step are spread evenly over its SLOTS slots: load i goes into slot i * SLOTS / N.  Calls `load` for those
// of slot S.
template <int S, int N, int SLOTS, class F>
__device__ __forceinline__ void loads_of_slot(F&& load) {
  static_for<0, N>([&](auto i) {
    if constexpr (decltype(i)::value * SLOTS / N == S) load(i);
  });
}

// K loop of the 16 x 16 x 32 form, operands loaded straight into LDS.  WHOLE: K is a whole number of 64-deep K
// tiles and the loads carry no range test; otherwise the chunks of the last K tile that lie past K are written
// as zeros (their offsets are pushed out of the buffer's range).  A K tile is two 32-deep steps of MB x NB MFMAs each, written as slots of
// four MFMAs plus one fragment read and at most one load (64-column tiles, whose K tile is bound by the bytes it waits
// for and not by issue: up to four reads and two loads).  All fragments of a step are read during the step
// before it, so a K tile's operands are no longer read once its second step starts: the barrier sits between
// the two steps.  LDS is a ring of P = 2D + 1 pieces (D = 2: five of 32 KiB; D = 3 and 4, 128-row tiles: seven
// and nine of 16 KiB); the A part of K tile j lives in piece 2j mod P and its B part in piece (2j + 1) mod P, so D and a
// half K tiles are resident:
//   step 0 of tile kt : fragment reads of step 1; loads of A(kt+D) into the piece idle since the last barrier
//   barrier           : every wave's part of tile kt+1 has landed, nobody reads tile kt any more
//   step 1 of tile kt : fragment reads of step 0 of tile kt+1; loads of B(kt+D) into the piece of A(kt)
// (T::TWO_RINGS: slots j mod (D + 1) of the A ring and j mod D of the B ring; A(kt+D) goes into the slot of A(kt-1), which is as
// idle as the piece of B(kt-1), and B(kt+D) into that of B(kt), as free after the barrier as the piece of A(kt))
// The loads go out one per two slots over the whole K tile and have one to three steps to land (with two
// whole-tile stages all of them went out during step 1 and had one to two: at operands that are not in the
// caches, cfg 2 and cfg 3 shapes beside the vendor GEMM, the ring takes 8-10 % less time; with operands that
// are, the same).
// An MFMA of this form holds the matrix pipe for 16 cycles and the wave is alone on its SIMD, so whatever is
// issued between two MFMAs has to fit into the 12 cycles the first one leaves: the read and the load of a slot
// go behind different MFMAs, each MFMA fenced so that the compiler keeps them there (measured: with both behind
// the slot's last MFMA the loads cost ~300 and the reads ~150 cycles of a K tile's 2048; spread like this the
// cfg 2 GEMM takes 4 % less time).
// On entry the LDS must be idle; on exit no load is in flight.  ROTATE: the K tiles are taken from k_first
// round to the one before it (see chiplet_k_tile; an instance of its own, since the counter costs the others 0.5 %).
template <class T, bool WHOLE, bool ROTATE, class ARow, class BRow>
__device__ __forceinline__ void gemm_mainloop_x16(typename T::Acc16& acc, const char* a_base, ARow a_row,
                                                     const char* b_base, BRow b_row, int K, char* lds, int k_first) {
  constexpr int MB = T::MB, NB = T::NB, READS = MB + T::B_READS * NB, AL = T::A_LOADS, BL = T::B_LOADS;
  constexpr int SLOTS = MB * NB / 4;   // per step
  constexpr int PIECE = T::PIECE_BYTES, D = T::DEPTH;
  static_assert(MB % 4 == 0 && READS <= 4 * SLOTS && (T::BN == 64 || (READS <= (T::B_KN ? 3 : 2) * SLOTS && AL <= SLOTS && BL <= SLOTS)),
                "at most two reads (B stored [K, N]: three) and one load per slot; 64 columns, whose K tile waits for its bytes: four and two");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave / 2, wn = wave % 2;
  const int lr = lane & 15, lq = lane >> 4;
  const int a_off = (wm * T::WTM + lr) * T::ROW_BYTES;
  int b_off[T::B_KN ? NB : 1];
  if constexpr (T::B_KN) {
    // inside its group of 16 lanes (k rows 8 lq .. + 3, + 4 with the second read), lane r points at k row r / 4, columns
    // 4 (r % 4) .. + 3 of the 16
    const int row = lq * 8 + (lr >> 2);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) b_off[nb] = row * T::PB + ((wn * NB + nb) ^ swz_kn<T::BN>(row)) * 32 + (lr & 3) * 8;
  } else {
    b_off[0] = (wn * T::WTN + lr) * T::ROW_BYTES;
  }
  int koff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) koff[ks] = ((ks * 4 + lq) ^ swz128_x16(lr)) * 16;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[nb][mb][v] = 0.f;

  const int kt_all = (K + 63) / 64;
  const int kt_last = kt_all - 1;
  Stager4W<T> st;
  st.init(a_base, a_row, b_base, b_row);
  auto wrap = [](int x) { return x >= T::PIECES ? x - T::PIECES : x; };
  char* const ring_b = T::TWO_RINGS ? lds + (D + 1) * T::A_BYTES : lds + PIECE;   // where B(0) lives
  constexpr int NEXT_A = T::TWO_RINGS ? T::A_BYTES : 2 * PIECE, NEXT_B = T::TWO_RINGS ? T::B_BYTES : 2 * PIECE;
  // load I of K tile kt into the piece at `piece` (the stager puts B loads T::A_BYTES behind the address it is given)
  auto load_a = [&](auto i, int kt, char* piece) { st.template issue_one<decltype(i)::value, WHOLE>(kt, K, piece); };
  auto load_b = [&](auto i, int kt, char* piece) { st.template issue_one<AL + decltype(i)::value, WHOLE>(kt, K, piece - T::A_BYTES); };
  int rotated = k_first;   // ROTATE: the K tile requested next
  auto next_rotated = [&] { rotated = rotated == kt_last ? 0 : rotated + 1; };
  static_for<0, D>([&](auto j) {
    constexpr int J = decltype(j)::value;
    const int kf = ROTATE ? rotated : min(J, kt_last);
    static_for<0, AL>([&](auto i) { load_a(i, kf, lds + J * NEXT_A); });
    static_for<0, BL>([&](auto i) { load_b(i, kf, ring_b + J * NEXT_B); });
    if constexpr (ROTATE) next_rotated();
  });
  wait_vmcnt<(D - 1) * (AL + BL)>();
  barrier_no_drain();
  Frags16<T> f0, f1;
  static_for<0, READS>([&](auto j) { read_one16<T, 0, decltype(j)::value>(f0, lds, ring_b, a_off, b_off, koff); });
  int ia = 0;   // piece of A(kt); TWO_RINGS: its slot
  int ib = 0;   // TWO_RINGS: slot of B(kt)
  for (int kt = 0; kt < kt_all; ++kt) {
    const char *cur_a, *cur_b, *nxt_a, *nxt_b;
    char *free_a, *free_b;
    if constexpr (T::TWO_RINGS) {
      cur_a = lds + ia * T::A_BYTES;
      cur_b = ring_b + ib * T::B_BYTES;
      free_a = lds + (ia == 0 ? D : ia - 1) * T::A_BYTES;   // held A(kt-1): nobody has read it since the last barrier
      free_b = ring_b + ib * T::B_BYTES;                    // B(kt): free after this iteration's barrier
      ia = ia == D ? 0 : ia + 1;
      ib = ib == D - 1 ? 0 : ib + 1;
      nxt_a = lds + ia * T::A_BYTES;
      nxt_b = ring_b + ib * T::B_BYTES;
    } else {
      cur_a = lds + ia * PIECE;
      cur_b = lds + wrap(ia + 1) * PIECE;
      nxt_a = lds + wrap(ia + 2) * PIECE;
      nxt_b = lds + wrap(ia + 3) * PIECE;
      free_a = lds + wrap(ia + 2 * D) * PIECE;   // held B(kt-1): nobody has read it since the last barrier
      free_b = lds + ia * PIECE;             // A(kt): free after this iteration's barrier
    }
    const int kf = ROTATE ? rotated : min(kt + D, kt_last);   // past the end some K tile is requested again, into pieces nobody reads
    static_for<0, SLOTS>([&](auto sl) {
      constexpr int S = decltype(sl)::value;
      mma_one16<T, S, 0>(acc, f0);
      if constexpr (S < READS) read_one16<T, 1, S>(f1, cur_a, cur_b, a_off, b_off, koff);
      __builtin_amdgcn_sched_barrier(0);
      mma_one16<T, S, 1>(acc, f0);
      if constexpr (SLOTS + S < READS) read_one16<T, 1, SLOTS + S>(f1, cur_a, cur_b, a_off, b_off, koff);
      __builtin_amdgcn_sched_barrier(0);
      mma_one16<T, S, 2>(acc, f0);
      if constexpr (3 * SLOTS + S < READS) read_one16<T, 1, 3 * SLOTS + S>(f1, cur_a, cur_b, a_off, b_off, koff);
      loads_of_slot<S, AL, SLOTS>([&](auto i) { load_a(i, kf, free_a); });
      __builtin_amdgcn_sched_barrier(0);
      mma_one16<T, S, 3>(acc, f0);
      if constexpr (2 * SLOTS + S < READS) read_one16<T, 1, 2 * SLOTS + S>(f1, cur_a, cur_b, a_off, b_off, koff);
      __builtin_amdgcn_sched_barrier(0);
    });
    wait_vmcnt<(D - 2) * (AL + BL) + AL>();   // this wave's part of tile kt+1 has landed (loads return in order); the younger ones may be in flight
    wait_lgkmcnt0();    // every read of tile kt has returned
    barrier_no_drain();
    static_for<0, SLOTS>([&](auto sl) {
      constexpr int S = decltype(sl)::value;
      mma_one16<T, S, 0>(acc, f1);
      if constexpr (S < READS) read_one16<T, 0, S>(f0, nxt_a, nxt_b, a_off, b_off, koff);
      __builtin_amdgcn_sched_barrier(0);
      mma_one16<T, S, 1>(acc, f1);
      if constexpr (SLOTS + S < READS) read_one16<T, 0, SLOTS + S>(f0, nxt_a, nxt_b, a_off, b_off, koff);
      __builtin_amdgcn_sched_barrier(0);
      mma_one16<T, S, 2>(acc, f1);
      if constexpr (3 * SLOTS + S < READS) read_one16<T, 0, 3 * SLOTS + S>(f0, nxt_a, nxt_b, a_off, b_off, koff);
      loads_of_slot<S, BL, SLOTS>([&](auto i) { load_b(i, kf, free_b); });
      __builtin_amdgcn_sched_barrier(0);
      mma_one16<T, S, 3>(acc, f1);
      if constexpr (2 * SLOTS + S < READS) read_one16<T, 0, 2 * SLOTS + S>(f0, nxt_a, nxt_b, a_off, b_off, koff);
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (!T::TWO_RINGS) ia = wrap(ia + 2);
    if constexpr (ROTATE) next_rotated();
  }
  wait_vmcnt0();   // the last iteration's requests are not left in flight
}

// ------------------------------------------------------------------ fp8 form
// K loop for e4m3 operands on v_mfma_f32_16x16x128_f8f6f4 (32 cycles, twice the flops per cycle and per byte of the
// bf16 instruction): a 128-byte K tile is one instruction deep, 8 x NB of them per wave.  LDS, loads, piece ring
// and the mid-tile barrier are those of gemm_mainloop_x16: the loop moves the same bytes per cycle of matrix work.
// A lane's 32 bytes of a fragment are the chunks lq and 4 + lq of its row (which k they are does not matter as long as
// both operands agree), so the reads are the conflict-free ones of the 16 x 16 x 32 form.
//
// A whole K tile of fragments is 128 registers, and holding two of them does not fit beside 256 accumulators.  The
// wave's quarter is therefore walked in four quadrants whose operand halves change one at a time:
//   Q0: a_lo x b_lo   reads b_hi            Q1: a_lo x b_hi   reads a_hi           (this K tile)
//   barrier: tile kt+1 has landed, nobody reads tile kt any more
//   Q2: a_hi x b_hi   reads a_lo of kt+1    Q3: a_hi x b_lo   reads b_lo of kt+1
// Every half is read one quadrant before its first use into registers that were last used the quadrant before; b_lo of
// the next tile lands in the registers of b_hi, so the two B halves change places from tile to tile (the loop body
// exists twice) and 128 fragment registers suffice with the reads spread evenly.
typedef int i32x8_t __attribute__((ext_vector_type(8)));

template <class T>
struct Frags8 {
  static constexpr int AH = T::MB / 2, BL = (T::NB + 1) / 2, BH = T::NB / 2;
  u32x4_t a[2][AH][2];   // [lo / hi rows][block][chunk lq, chunk 4 + lq]
  u32x4_t b[2][BL][2];   // [register set]: b_lo of the tiles of parity P is set P, b_hi set 1 - P
};

__device__ __forceinline__ i32x8_t join_f8(const u32x4_t lo, const u32x4_t hi) {
  return __builtin_bit_cast(i32x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// which of the `n` events spread over the first `slots` slots belongs to slot s (-1: none)
constexpr int event_in_slot(int s, int n, int slots) {
  for (int i = 0; i < n; ++i)
    if (i * slots / n == s) return i;
  return -1;
}

// On entry the LDS must be idle; on exit no load is in flight.
template <class T, bool WHOLE, class ARow, class BRow>
__device__ __forceinline__ void gemm_mainloop_f8(typename T::Acc16& acc, const char* a_base, ARow a_row,
                                                    const char* b_base, BRow b_row, int K, char* lds) {
  typedef Frags8<T> F;
  constexpr int AL = T::A_LOADS, BLD = T::B_LOADS, PIECE = T::A_BYTES;
  constexpr int AH = F::AH, NL = F::BL, NH = F::BH;
  constexpr int HALF_MMAS = AH * T::NB;   // matrix instructions between two events of the barrier
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave / 2, wn = wave % 2;
  const int lr = lane & 15, lq = lane >> 4;
  const int a_off = (wm * T::WTM + lr) * T::ROW_BYTES;
  const int b_off = (wn * T::WTN + lr) * T::ROW_BYTES;
  int koff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) koff[ks] = ((ks * 4 + lq) ^ swz128_x16(lr)) * 16;
#pragma unroll
  for (int nb = 0; nb < T::NB; ++nb)
#pragma unroll
    for (int mb = 0; mb < T::MB; ++mb) acc[nb][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int kt_all = (K + 63) / 64;
  const int kt_last = kt_all - 1;
  Stager4W<T> st;
  st.init(a_base, a_row, b_base, b_row);
  auto wrap = [](int x) { return x >= 5 ? x - 5 : x; };
  auto load_a = [&](auto i, int kt, char* piece) { st.template issue_one<decltype(i)::value, WHOLE>(kt, K, piece); };
  auto load_b = [&](auto i, int kt, char* piece) { st.template issue_one<AL + decltype(i)::value, WHOLE>(kt, K, piece - T::A_BYTES); };
  static_for<0, AL>([&](auto i) { load_a(i, 0, lds); });
  static_for<0, BLD>([&](auto i) { load_b(i, 0, lds + PIECE); });
  static_for<0, AL>([&](auto i) { load_a(i, min(1, kt_last), lds + 2 * PIECE); });
  static_for<0, BLD>([&](auto i) { load_b(i, min(1, kt_last), lds + 3 * PIECE); });
  wait_vmcnt<AL + BLD>();
  barrier_no_drain();

  F f;
  // read J of a half: block J / 2, chunk J % 2
  auto read_a = [&](auto j, auto half, const char* piece) {
    constexpr int J = decltype(j)::value, H = decltype(half)::value;
    f.a[H][J / 2][J % 2] = *(const u32x4_t*)(piece + a_off + (H * AH + J / 2) * 16 * 128 + koff[J % 2]);
  };
  auto read_b = [&](auto j, auto set, auto first, const char* piece) {
    constexpr int J = decltype(j)::value, S = decltype(set)::value, FIRST = decltype(first)::value;
    f.b[S][J / 2][J % 2] = *(const u32x4_t*)(piece + b_off + (FIRST + J / 2) * 16 * 128 + koff[J % 2]);
  };
  using std::integral_constant;
  typedef integral_constant<int, 0> I0;
  typedef integral_constant<int, 1> I1;
  static_for<0, 2 * AH>([&](auto j) { read_a(j, I0{}, lds); });
  static_for<0, 2 * NL>([&](auto j) { read_b(j, I0{}, I0{}, lds + PIECE); });

  int ia = 0;   // piece of A(kt)
  auto tile = [&](auto parity, int kt) {
    constexpr int P = decltype(parity)::value;
    const char* cur_a = lds + ia * PIECE;
    const char* cur_b = lds + wrap(ia + 1) * PIECE;
    const char* nxt_a = lds + wrap(ia + 2) * PIECE;
    const char* nxt_b = lds + wrap(ia + 3) * PIECE;
    char* free_a = lds + wrap(ia + 4) * PIECE;   // held B(kt-1): nobody has read it since the last barrier
    char* free_b = lds + ia * PIECE;             // A(kt): free after this iteration's barrier
    const int kf = min(kt + 2, kt_last);         // past the end the last K tile is requested again, into pieces nobody reads
    // one quadrant: rows of half AHALF, columns of half BHALF; ROWS_OUTER: the A half is the newer one, its last block
    // is used last.  BASE: matrix instructions of this barrier interval before the quadrant (which loads are due).
    auto quadrant = [&](auto ahalf, auto bhalf, auto rows_outer, auto reads, auto window, auto base, auto read, auto nloads, auto load) {
      constexpr int A = decltype(ahalf)::value, BH_ = decltype(bhalf)::value;
      constexpr bool RO = decltype(rows_outer)::value != 0;
      constexpr int NBQ = BH_ ? NH : NL, N = AH * NBQ, R = decltype(reads)::value, W = decltype(window)::value + N;
      constexpr int SET = BH_ ? 1 - P : P;
      static_for<0, N>([&](auto sl) {
        constexpr int S = decltype(sl)::value;
        constexpr int mb = RO ? S / NBQ : S % AH, nb = RO ? S % NBQ : S / AH;
        f32x4_t& c = acc[BH_ * NL + nb][A * AH + mb];
        c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(join_f8(f.b[SET][nb][0], f.b[SET][nb][1]),
                                                             join_f8(f.a[A][mb][0], f.a[A][mb][1]), c, 0, 0, 0, 0, 0, 0);
        constexpr int rd = event_in_slot(S, R, W);
        if constexpr (rd >= 0) read(integral_constant<int, (rd >= 0 ? rd : 0)>{});
        constexpr int ld = event_in_slot(decltype(base)::value + S - 1, decltype(nloads)::value, HALF_MMAS);   // not behind the same instruction as a read
        if constexpr (ld >= 0) load(integral_constant<int, (ld >= 0 ? ld : 0)>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    typedef integral_constant<int, -4> Early;    // reads done four instructions before the quadrant ends: the barrier waits for them
    quadrant(I0{}, I0{}, I0{}, integral_constant<int, 2 * NH>{}, I0{}, I0{},
             [&](auto j) { read_b(j, integral_constant<int, 1 - P>{}, integral_constant<int, NL>{}, cur_b); },
             integral_constant<int, AL>{}, [&](auto i) { load_a(i, kf, free_a); });
    quadrant(I0{}, I1{}, I0{}, integral_constant<int, 2 * AH>{}, Early{}, integral_constant<int, AH * NL>{},
             [&](auto j) { read_a(j, I1{}, cur_a); },
             integral_constant<int, AL>{}, [&](auto i) { load_a(i, kf, free_a); });
    wait_vmcnt<AL>();   // this wave's part of tile kt+1 has landed (loads return in order); A(kt+2) may be in flight
    wait_lgkmcnt0();    // every read of tile kt has returned
    barrier_no_drain();
    quadrant(I1{}, I1{}, I1{}, integral_constant<int, 2 * AH>{}, I0{}, I0{},
             [&](auto j) { read_a(j, I0{}, nxt_a); },
             integral_constant<int, BLD>{}, [&](auto i) { load_b(i, kf, free_b); });
    quadrant(I1{}, I0{}, I1{}, integral_constant<int, 2 * NL>{}, I0{}, integral_constant<int, AH * NH>{},
             [&](auto j) { read_b(j, integral_constant<int, 1 - P>{}, I0{}, nxt_b); },
             integral_constant<int, BLD>{}, [&](auto i) { load_b(i, kf, free_b); });
    ia = wrap(ia + 2);
  };
  for (int kt = 0; kt < kt_all; kt += 2) {
    tile(I0{}, kt);
    if (kt + 1 < kt_all) tile(I1{}, kt + 1);
  }
  wait_vmcnt0();   // the last iteration's requests (the last K tile once more) are not left in flight
}

// One barrier per 64-deep K tile.  A single wave per SIMD has to keep the matrix pipe fed
// while it also issues every memory instruction, so the loop body is written as slots of two
// MFMAs plus a few memory instructions, each slot fenced so that the compiler keeps the
// interleaving (four 16-deep steps ks0..ks3 of PAIRS slots each):
//   steps ks0, ks1 of tile kt : fragments of the next step; LDS stores of tile kt+1
//   step  ks2                : fragments of ks3 (in its first half)
//   barrier
//   step  ks3                : first fragments of tile kt+1 (in its first half)
//   every other slot         : global loads of tile kt+2, each after the LDS store that frees
//                               its register
// The body is branch-free (past the end the last tile is staged again into a free stage).
// On entry the LDS stages must be idle (every wave of the work-group past its last access to them): they are written
// from the first instruction on.  On exit none of the wave's loads
// is in flight; other waves may still be reading fragments, so a barrier precedes any reuse of the stages.
template <class T, bool ROTATE = false, class ARow, class BRow>
__device__ __forceinline__ void gemm_mainloop(typename T::Acc& acc, const char* a_base, ARow a_row,
                                                 const char* b_base, BRow b_row, int K, char* lds, int k_first = 0) {
  if constexpr (T::F8) {
    if (K % 64 == 0) gemm_mainloop_f8<T, true>(acc, a_base, a_row, b_base, b_row, K, lds);
    else gemm_mainloop_f8<T, false>(acc, a_base, a_row, b_base, b_row, K, lds);
    return;
  } else if constexpr (T::X16) {
    // two copies of the loop: the per-load range test of a ragged last K tile costs the others 0.8 %
    if (K % 64 == 0) gemm_mainloop_x16<T, true, ROTATE>(acc, a_base, a_row, b_base, b_row, K, lds, k_first);
    else gemm_mainloop_x16<T, false, ROTATE>(acc, a_base, a_row, b_base, b_row, K, lds, k_first);
    return;
  } else {
  constexpr int PAIRS = T::PAIRS, SLOTS = T::SLOTS, READS = T::READS, LOADS = T::LOADS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave / 2, wn = wave % 2;
  const int lr = lane & 31, lh = lane >> 5;
  const int a_off = (wm * T::WTM + lr) * T::ROW_BYTES;
  const int b_off = T::A_BYTES + (wn * T::WTN + lr) * T::ROW_BYTES;
  int koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) koff[ks] = ((ks * 2 + lh) ^ swz128(lr)) * 16;
#pragma unroll
  for (int ni = 0; ni < T::NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < T::MI; ++mi)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[ni][mi][v] = 0.f;

  const int kt_all = (K + 63) / 64;
  const int kt_last = kt_all - 1;
  Stager4W<T> st;
  st.init(a_base, a_row, b_base, b_row);
  // the first two K tiles are requested together (the second into registers that are free until the
  // loop starts), so the tile pays for one cold round trip to memory, not two in a row
  st.template fetch_range<0, LOADS>(0, K);
  u32x4_t second[LOADS];
  static_for<0, LOADS>([&](auto i) { second[decltype(i)::value] = st.template load_one<decltype(i)::value>(min(1, kt_last), K); });
  st.template commit_range<0, LOADS>(lds);
  static_for<0, LOADS>([&](auto i) { st.reg[decltype(i)::value] = second[decltype(i)::value]; });
  __syncthreads();

  Frags4W<T> f0, f1;
  read_range<T, 0, 0, READS>(f0, lds, a_off, b_off, koff);
  for (int kt = 0; kt < kt_all; ++kt) {
    const char* cur = lds + (kt & 1) * T::STAGE_BYTES;
    char* nxt = lds + ((kt + 1) & 1) * T::STAGE_BYTES;
    const int kf = min(kt + 2, kt_last);
    static_for<0, SLOTS>([&](auto sl) {
      constexpr int S = decltype(sl)::value, PART = S / PAIRS, J = S % PAIRS;
      if constexpr (S == 3 * PAIRS) {
        wait_lgkmcnt0();   // own LDS stores of tile kt+1 are done and every read of tile kt has returned
        barrier_no_drain();
      }
      mma_pair<T, J>(acc, (PART & 1) ? f1 : f0);
      // fragment reads: one step ahead, spread over the step's slots; the steps around the barrier
      // read in their first half so that the waits find the data there
      if constexpr (PART == 0) read_range<T, 1, J * READS / PAIRS, (J + 1) * READS / PAIRS>(f1, cur, a_off, b_off, koff);
      if constexpr (PART == 1) read_range<T, 2, J * READS / PAIRS, (J + 1) * READS / PAIRS>(f0, cur, a_off, b_off, koff);
      if constexpr (PART == 2 && J < T::HALF)
        read_range<T, 3, J * READS / T::HALF, (J + 1) * READS / T::HALF>(f1, cur, a_off, b_off, koff);
      if constexpr (PART == 3 && J < T::HALF)
        read_range<T, 0, J * READS / T::HALF, (J + 1) * READS / T::HALF>(f0, nxt, a_off, b_off, koff);
      // register i goes to LDS during the first two steps and is refilled (tile kt+2) later in
      // the iteration: the loads are spread over the whole iteration, since a burst would
      // saturate the address unit and stall the wave
      if constexpr (S < 2 * PAIRS) st.template commit_range<S * LOADS / (2 * PAIRS), (S + 1) * LOADS / (2 * PAIRS)>(nxt);
      if constexpr (S % 2 == 1) st.template fetch_range<(S / 2) * LOADS / (SLOTS / 2), (S / 2 + 1) * LOADS / (SLOTS / 2)>(kf, K);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  }
}

// Mainloop over a ring of NST stages filled by direct-to-LDS loads, NST - 1 K tiles ahead, one barrier per K tile, for a
// work-group of eight waves: waves 0-3 (one per SIMD) only read fragments and issue MFMAs, waves 4-7 only issue the loads.
// A wave issues in order, so the load instructions of a K tile and its matrix work would otherwise follow one another.
// Requests past the last K tile are out of the buffers' range: zeros are written, memory is not asked.  Returns true in the
// computing waves (which hold the accumulators) and false in the loading waves, whose requests have all completed.
template <class T, int NST, class ARow, class BRow>
__device__ __forceinline__ bool gemm_mainloop_ring_split(typename T::Acc32& acc, const char* a_base, ARow a_row,
                                                            const char* b_base, BRow b_row, int K, char* lds) {
  static_assert(T::DIRECT && !T::B_KN, "ring staging is written for [N, K] operands loaded straight into LDS");
  constexpr int PAIRS = T::PAIRS, READS = T::READS, LOADS = T::LOADS;
  static_assert((NST - 2) * LOADS <= 63 && NST >= 3, "wait-count immediate");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int kt_all = (K + 63) / 64;
  if (wave >= T::NWAVES) {
    Stager4W<T> st;
    st.init(a_base, a_row, b_base, b_row, (int)threadIdx.x - T::THREADS);
#pragma unroll
    for (int j = 0; j < NST - 1; ++j) st.template issue_range<0, LOADS>(j, K, lds + j * T::STAGE_BYTES);
#pragma unroll 1
    for (int kt = 0; kt < kt_all; ++kt) {
      wait_vmcnt<(NST - 2) * LOADS>();   // this wave's part of tile kt has landed (loads return in order)
      barrier_no_drain();                // ... everybody's, and the computing waves are past tile kt - 1
      st.template issue_range<0, LOADS>(kt + NST - 1, K, lds + ((kt + NST - 1) % NST) * T::STAGE_BYTES);
    }
    wait_vmcnt0();
    return false;
  }
  const int wm = wave / 2, wn = wave % 2;
  const int lr = lane & 31, lh = lane >> 5;
  const int a_off = (wm * T::WTM + lr) * T::ROW_BYTES;
  const int b_off = T::A_BYTES + (wn * T::WTN + lr) * T::ROW_BYTES;
  int koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) koff[ks] = ((ks * 2 + lh) ^ swz128(lr)) * 16;
#pragma unroll
  for (int ni = 0; ni < T::NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < T::MI; ++mi)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[ni][mi][v] = 0.f;
#pragma unroll 1
  for (int kt = 0; kt < kt_all; ++kt) {
    barrier_no_drain();
    const char* cur = lds + (kt % NST) * T::STAGE_BYTES;
    Frags4W<T> f0, f1;
    read_range<T, 0, 0, READS>(f0, cur, a_off, b_off, koff);
    read_range<T, 1, 0, READS>(f1, cur, a_off, b_off, koff);
    static_for<0, PAIRS>([&](auto j) { mma_pair<T, decltype(j)::value>(acc, f0); });
    read_range<T, 2, 0, READS>(f0, cur, a_off, b_off, koff);
    static_for<0, PAIRS>([&](auto j) { mma_pair<T, decltype(j)::value>(acc, f1); });
    read_range<T, 3, 0, READS>(f1, cur, a_off, b_off, koff);
    static_for<0, PAIRS>([&](auto j) { mma_pair<T, decltype(j)::value>(acc, f0); });
    static_for<0, PAIRS>([&](auto j) { mma_pair<T, decltype(j)::value>(acc, f1); });
    wait_lgkmcnt0();   // every read of tile kt has returned before the next barrier frees its stage
  }
  return true;
}

// Epilogue: each wave turns its accumulators into bf16, parks them in its
// own piece of the (now idle) operand stages, and reads them back row by row so that every
// global store covers whole 128-byte lines (one row = WTN bf16 = SL slots of 16 bytes, read by
// SL lanes; written straight from the MFMA layout, a store instruction would scatter 8-byte
// pieces over 32 rows).  A parked row has SLP >= SL slots (a power of two); the 16-byte slot g
// of row m lives at slot g ^ key(m), which keeps the 8-byte writes (2-way at worst) and the
// 16-byte reads away from bank conflicts.  THROUGH: the global stores are written through (for a tile that a flag or
// counter announces: see stores_done).
template <class T>
struct ParkedTile {
  static constexpr int SL = T::WTN / 8;            // 16-byte slots of data per row: 16, 12 or 8
  static constexpr int SLP = SL <= 8 ? 8 : 16;     // slots per parked row
  static constexpr int ROW = SLP * 16;             // bytes per parked row
  static_assert(4 * T::WTM * ROW <= T::LDS_BYTES, "the parked tile fits in the operand stages");
  // 128-byte rows pair up in a 256-byte bank window
  __device__ static __forceinline__ int key(int m) { return SLP == 16 ? (m & 15) : ((m >> 1) & 7); }
};

// No scales: every factor is one.
struct Unscaled {};

// First half of the epilogue: accumulators -> bf16 -> the wave's piece of the operand stages.  `scales` (16 x 16 blocks
// only): row(r) and cols(c) give the factors of the tile's row r and of its columns c .. c + 3; a value becomes
// (value * row) * column before it is rounded.
template <class T, class Scales = Unscaled>
__device__ __forceinline__ void park_tile_bf16(const typename T::Acc& acc, char* lds, Scales scales = Scales{}) {
  typedef ParkedTile<T> P;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  __syncthreads();   // every wave is done reading the operand stages
  char* park = lds + wave * (T::WTM * P::ROW);
  if constexpr (T::X16) {
    // a lane holds, per block, row (lane % 16) and the four columns 4 (lane / 16) .. + 3: half a 16-byte slot
    const int lr = lane & 15, lq = lane >> 4;
    auto park_block = [&](int mb, int nb, const f32x4_t x) {
      const int m = mb * 16 + lr, g = nb * 2 + (lq >> 1);
      bf16x4_t v = {(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
      *(bf16x4_t*)(park + m * P::ROW + ((g ^ P::key(m)) * 16) + (lq & 1) * 8) = v;
    };
    if constexpr (std::is_same_v<Scales, Unscaled>) {
#pragma unroll
      for (int mb = 0; mb < T::MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < T::NB; ++nb) park_block(mb, nb, acc[nb][mb]);
    } else {
      const int wm = wave / T::WAVES_N, wn = wave % T::WAVES_N;
      float rs[T::MB];
#pragma unroll
      for (int mb = 0; mb < T::MB; ++mb) rs[mb] = scales.row(wm * T::WTM + mb * 16 + lr);
#pragma unroll
      for (int nb = 0; nb < T::NB; ++nb) {
        const f32x4_t cs = scales.cols(wn * T::WTN + nb * 16 + lq * 4);
#pragma unroll
        for (int mb = 0; mb < T::MB; ++mb) park_block(mb, nb, acc[nb][mb] * rs[mb] * cs);
        __builtin_amdgcn_sched_barrier(0);   // a column block at a time: its values, not the whole tile's, are in registers
      }
    }
    wait_lgkmcnt0();
    return;
  } else {
  const int lr = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int mi = 0; mi < T::MI; ++mi) {
    const int m = mi * 32 + lr;
#pragma unroll
    for (int ni = 0; ni < T::NI; ++ni) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int g = ni * 4 + q;
        bf16x4_t v = {(__bf16)acc[ni][mi][q * 4 + 0], (__bf16)acc[ni][mi][q * 4 + 1],
                      (__bf16)acc[ni][mi][q * 4 + 2], (__bf16)acc[ni][mi][q * 4 + 3]};
        *(bf16x4_t*)(park + m * P::ROW + ((g ^ P::key(m)) * 16) + lh * 8) = v;
      }
    }
  }
  // the reads that follow are the same wave's: LDS operations of one wave complete in order
  wait_lgkmcnt0();
  }
}

// Second half: the rows m_lo <= m < m_hi of the parked tile (global row numbers; the tile starts at row
// m0, column n0) go to c[m, n] with leading dimension ldc.  May be called several times with different
// windows and destinations.
template <class T, bool THROUGH = false>
__device__ __forceinline__ void store_parked_bf16(__bf16* c, size_t ldc, int m0, int n0, int m_lo, int m_hi, int N,
                                                      const char* lds) {
  typedef ParkedTile<T> P;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave / 2, wn = wave % 2;
  const char* park = lds + wave * (T::WTM * P::ROW);
  constexpr int ROWS_PER_READ = 64 / P::SLP;
  const int g = lane % P::SLP;
  const int gn = n0 + wn * T::WTN + g * 8;
  __bf16* wave_c = c + (size_t)(m0 + wm * T::WTM) * ldc;
  // 32-bit offsets reach over all rows of the wave up to 2^22 columns; beyond, the base moves with the rows
  const bool wide = ldc > (1u << 22);
  const __amdgpu_buffer_rsrc_t all_rows = __builtin_amdgcn_make_buffer_rsrc((void*)wave_c, 0, -1, 0x00020000);
#pragma unroll 8
  for (int it = 0; it < T::WTM / ROWS_PER_READ; ++it) {
    const int row = it * ROWS_PER_READ + lane / P::SLP;
    const u32x4_t v = *(const u32x4_t*)(park + row * P::ROW + ((g ^ P::key(row)) * 16));
    const int gm = m0 + wm * T::WTM + row;
    if (g < P::SL && gm >= m_lo && gm < m_hi && gn < N) {
      if constexpr (THROUGH) {
        if (wide) {
          const __amdgpu_buffer_rsrc_t rows =
              __builtin_amdgcn_make_buffer_rsrc((void*)(wave_c + (size_t)(it * ROWS_PER_READ) * ldc), 0, -1, 0x00020000);
          __builtin_amdgcn_raw_buffer_store_b128(v, rows, (int)(((uint32_t)(lane / P::SLP) * (uint32_t)ldc + (uint32_t)gn) * 2u), 0, kThrough);
        } else {
          __builtin_amdgcn_raw_buffer_store_b128(v, all_rows, (int)(((uint32_t)row * (uint32_t)ldc + (uint32_t)gn) * 2u), 0, kThrough);
        }
      }
      else *(u32x4_t*)(c + (size_t)gm * ldc + gn) = v;
    }
  }
}

template <class T, bool THROUGH = false>
__device__ __forceinline__ void store_tile_bf16(const typename T::Acc& acc, __bf16* c, size_t ldc, int m0,
                                                    int n0, int M, int N, char* lds) {
  park_tile_bf16<T>(acc, lds);
  store_parked_bf16<T, THROUGH>(c, ldc, m0, n0, m0, M, N, lds);
}

}  // namespace ditron
