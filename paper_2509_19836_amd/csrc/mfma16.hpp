// Building blocks on v_mfma_f32_16x16x32_bf16 with LDS tiles filled by direct global -> LDS loads.
//
// Register layouts (lane l: r = l % 16, g = l / 16):
//   A operand (M x K): lane holds A[m = r][k = 8g .. 8g+7]
//   B operand (K x N): lane holds B[k = 8g .. 8g+7][n = r]
//   C/D (M x N), 4 fp32: register v holds C[m = 4g + v][n = r]
// Two accumulator tiles whose M indices are the next contraction index (rows 32c .. 32c+15 and 32c+16 ..
// 32c+31) packed to bf16 side by side are the B operand of that contraction: element e of lane (r, g) is row
// 32c + 16 (e / 4) + 4g + e % 4, and the A operand only has to be read in the same row order (cols_operand).
//
// LDS tiles are row-major [rows][D] bf16 without padding (a direct load writes 1 KiB of consecutive LDS per
// wave), the 16-byte chunks of a row permuted by chunk ^ swz(row), which moves pairs of chunks: the 32-byte
// pieces that half a wave takes from 8 rows in a transposing read fall into 8 different places of the 256-byte
// bank line, and the chunks of the row-wise read (16 lanes at a time, four-lane groups of g and g + 1 that never
// name rows 8 apart with the same g) into 16 different ones.
#pragma once
#include "common.hpp"

namespace burst {

typedef __attribute__((address_space(3))) char* lds_bytes;

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

template <int D>
__device__ __forceinline__ int swz(int row) {   // depends on row % 16 only
  static_assert(D == 64 || D == 128, "row of 8 or 16 chunks");
  return D == 128 ? (row & 7) << 1 : ((row >> 1) & 3) << 1;
}

// LDS byte offsets of a lane's operand reads inside a tile of D columns.  Adding multiples of 16 rows keeps them;
// the k-step or column block is one exclusive or (swz moves pairs of chunks, so it commutes with both).
template <int D>
struct OperandAddr {
  uint32_t rows;   // k-step 0: row r, columns 8g .. +7
  uint32_t cols;   // column block 0: this lane's 8 bytes of the transposing read of rows 4g + r / 4
  __device__ __forceinline__ void init(int lane) {
    const int r = lane & 15, g = lane >> 4, row = 4 * g + (r >> 2);
    rows = r * 2 * D + ((g ^ swz<D>(r)) << 4);
    cols = row * 2 * D + ((((r & 3) >> 1) ^ swz<D>(row)) << 4) + 8 * (r & 1);
  }
};

// Operand with lane = tile row: rows row0 + r (row0 a multiple of 16), columns 32 ks + 8g .. +7.  `tile`: LDS byte
// address of the tile, a multiple of 256.
template <int D>
__device__ __forceinline__ bf16x8 rows_operand(uint32_t tile, const OperandAddr<D>& ad, int row0, int ks) {
  const lds_bytes p = (lds_bytes)(uintptr_t)((tile + ad.rows) ^ (uint32_t)(64 * ks));
  return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(p + row0 * 2 * D);
}
// Operand with lane = tile column 16 db + r, the 32 rows row0 .. row0 + 31 in packed-accumulator order.
template <int D>
__device__ __forceinline__ bf16x8 cols_operand(uint32_t tile, const OperandAddr<D>& ad, int row0, int db) {
  typedef __attribute__((address_space(3))) s16x4* tr_ptr;
  const lds_bytes p = (lds_bytes)(uintptr_t)((tile + ad.cols) ^ (uint32_t)(32 * db));
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(p + row0 * 2 * D));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(p + (row0 + 16) * 2 * D));
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, both);
}

// Packed B operand from two accumulator tiles (rows 0..15 and 16..31 of the 32-row chunk).  The empty assembly
// statement keeps the conversions where they are written: the compiler otherwise moves them behind the next
// barrier, into another phase.
__device__ __forceinline__ bf16x8 pack_pair(const f32x4& lo, const f32x4& hi) {
  bf16x8 x = {(__bf16)lo[0], (__bf16)lo[1], (__bf16)lo[2], (__bf16)lo[3],
              (__bf16)hi[0], (__bf16)hi[1], (__bf16)hi[2], (__bf16)hi[3]};
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ bf16x8 zero_operand() {
  const u32x4 z = {0, 0, 0, 0};
  return __builtin_bit_cast(bf16x8, z);
}

// One direct load: every lane's 16 bytes at base + offset go to LDS at lds + 16 * lane.  Written as an
// assembly statement because the compiler otherwise waits for all of them before the next LDS read; the
// kernels wait by count themselves (wait_loads_barrier).  m0 is a reserved register, which the compiler keeps no
// value in; nothing else in these kernels uses it.
// The compiler does not look for hazards inside the statement.  A load that goes to LDS needs one wait state behind a scalar
// write of m0, the s_nop (with four, each up to four clocks between two MFMAs: dQ 2423 us instead of 2399, dK/dV 3428 instead of
// 3377; 16384 rows, 32 heads, d = 128).  And it must stay five behind a vector instruction that wrote its address, as
// v_readfirstlane_b32 or the return of a spilled scalar register from a lane do; the statement has two.  The addresses come from
// scalar arithmetic, and the build refuses a kernel in which one does not (build.check_load_addresses).  A scalar copy of the
// address in place of the s_nop would do without the check, at 0.3-0.5 % of a case.
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t offset, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory");
}
// The same with 4 bytes per lane.
__device__ __forceinline__ void load_dword_to_lds(const char* base, uint32_t offset, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory");
}
// Wait until at most N of this wave's global loads are outstanding, then meet the other waves.  Work-group
// barrier without the full drain of __syncthreads: loads of later tiles stay in flight.  The scheduling fences
// keep arithmetic, which the memory clobber does not bind, from drifting across.
template <int N>
__device__ __forceinline__ void wait_loads_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// The same wait without the meeting, for tiles that a wave brings for itself.
template <int N>
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// The same meeting without waiting for loads: between two phases of a wave.
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// The same with all but the last N of this wave's LDS instructions done (they complete in order): for a phase whose
// stores the other half reads, followed by N LDS reads for the next phase, which stay in flight.
template <int N>
__device__ __forceinline__ void stores_barrier() {
  static_assert(N <= 15, "lgkmcnt has four bits");
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// The same and all of this wave's global loads done.
template <int N>
__device__ __forceinline__ void stores_loads_barrier() {
  static_assert(N <= 15, "lgkmcnt has four bits");
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// Nothing moves across: the LDS stores that stores_barrier counts on stay in front of the reads it leaves in flight.
__device__ __forceinline__ void keep_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Keeps the computation of a wave-uniform value where it is written.  The compiler sinks scalar arithmetic to its use, for
// a loop-carried value the head of the next iteration: there it stood between a barrier and the first MFMA of a matrix
// phase (35-40 instructions, in which no wave of the SIMD has matrix work) instead of behind MFMAs.  16384 rows, 32 heads,
// d = 128: dK/dV 3769 -> 3438 us, dQ 2425 -> 2400, forward 1769 -> 1733; in forward, whose vector phase is the longer one, the
// rest of that work is better off at the head of the matrix phase (moved into the vector phase: 1796).
template <class T>
__device__ __forceinline__ void pin(T& x) {
  asm volatile("" : "+s"(x));
}
template <class T, class... Rest>
__device__ __forceinline__ void pin(T& x, Rest&... rest) {
  pin(x);
  pin(rest...);
}

// Any value.  Registers that a walk fills before it reads them, on paths the compiler cannot tell, are otherwise carried
// around the loop over the steps as values it might need (a hundred of them in the dQ kernel, which then spilled).
template <class T, int M, int N>
__device__ __forceinline__ void any_value(T (&x)[M][N]) {
#pragma unroll
  for (int i = 0; i < M * N; ++i) asm volatile("" : "=v"(x[i / N][i % N]));
}
template <class T, int N>
__device__ __forceinline__ void any_value(T (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "=v"(x[i]));
}

// All ones where x is negative, else zero: scalar arithmetic in place of conditions, minima and maxima, whose results the
// compiler keeps in vector registers.
__device__ __forceinline__ int negative_mask(int x) {
  pin(x);   // (it would recognise the condition)
  return x >> 31;
}

// Direct staging of [ROWS x D] tiles by NW waves: wave w brings 1 KiB pieces w, w + NW, ...  The per-lane part
// of an address is a 32-bit offset computed once, the first row of the tile is a wave-uniform pointer.
template <int D, int ROWS, int NW>
struct DirectStager {
  static constexpr int PITCH = 2 * D, RPI = 1024 / PITCH;        // rows per load instruction
  static constexpr int BYTES = ROWS * PITCH, N = BYTES / 1024 / NW;   // loads per wave
  static_assert(N * NW * 1024 == BYTES, "whole pieces per wave");
  uint32_t off[N];
  __device__ __forceinline__ int row_of(int i, int wave, int lane) const { return (i * NW + wave) * RPI + lane / (PITCH / 16); }
  __device__ __forceinline__ uint32_t offset(int row, int lane_row, int64_t ss, int lane) const {
    uint32_t x = 2u * ((uint32_t)row * (uint32_t)ss + (uint32_t)(((lane % (PITCH / 16)) ^ swz<D>(lane_row)) * 8));
    asm("" : "+v"(x));   // (a product's low half otherwise keeps a pair of registers)
    return x;
  }
  __device__ __forceinline__ void init(int64_t ss, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i) off[i] = offset(row_of(i, wave, lane), row_of(i, wave, lane), ss, lane);
  }
  __device__ __forceinline__ void load_one(const char* tile, int i, uint32_t lds, int wave) const {
    load_to_lds(tile, off[i], lds + (i * NW + wave) * 1024);
  }
  // for a tile that reaches past the last row: rows beyond `valid` - 1 are read as copies of that row
  __device__ __forceinline__ void clamp(int64_t ss, int valid, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i) off[i] = offset(min(row_of(i, wave, lane), valid - 1), row_of(i, wave, lane), ss, lane);
  }
};

// The same by one wave alone, whose many loads of a tile would need a register each.  Eight rows of a tile after the other have the
// same offsets from their first one (swz has that period): KEEP_ALL false holds those of eight rows only.
template <int D, int ROWS, bool KEEP_ALL>
struct WaveStager {
  using Each = DirectStager<D, ROWS, 1>;
  static constexpr int N = Each::N, PER = KEEP_ALL ? N : 8 / Each::RPI;   // loads of a tile; offsets
  uint32_t off[PER];
  static __device__ __forceinline__ uint32_t offset(int i, int last, int64_t ss, int lane) {
    const int row = Each().row_of(i, 0, lane);
    return Each().offset(min(row, last), row, ss, lane);
  }
  __device__ __forceinline__ void init(int64_t ss, int lane) {
#pragma unroll
    for (int i = 0; i < PER; ++i) off[i] = offset(i, ROWS, ss, lane);
  }
  // rows of the tile beyond `valid` - 1 are read as copies of that one
  __device__ __forceinline__ void load(const char* tile, int64_t ss, int valid, uint32_t lds, int lane) const {
    if (valid >= ROWS) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        load_to_lds(tile, off[i % PER], lds + i * 1024);
        if (i % PER == PER - 1) {
          tile += 2 * PER * Each::RPI * ss;
          pin(tile);
        }
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) load_to_lds(tile, offset(i, valid - 1, ss, lane), lds + i * 1024);
  }
};

// The tiles of the walked axis that a block-wise sparse mask leaves open, in order: the flags of 64 tiles at a time as bits
// of a scalar register, one LDS read for each 64 tiles of the axis.
struct OpenTiles {
  const uint8_t* flags;   // LDS, kMaxBlockCacheTiles of them
  uint64_t bits;          // of tiles base .. base + 63: open and not handed out yet
  int base;
  __device__ __forceinline__ void read() { bits = __ballot(flags[base + (threadIdx.x & 63)] != 0); }
  // From `tile` on
  __device__ __forceinline__ void start(int tile) {
    base = tile & ~63;
    read();
    bits &= ~0ull << (tile & 63);
  }
  // The next open tile below `end` (at most kMaxBlockCacheTiles), -1 when there is none
  __device__ __forceinline__ int next(int end) {
    while (bits == 0) {
      base += 64;
      if (base >= end) return -1;
      read();
    }
    const int tile = base + __builtin_ctzll(bits);
    bits &= bits - 1;
    return __builtin_amdgcn_readfirstlane(tile < end ? tile : -1);
  }
};

// Walk of a query block over the key tiles (BK rows) it can see.  The visible tiles are one run of consecutive
// tiles, so the cursor and the tile addresses move by adding constants.  Tiles are brought in sets:
// {K of tile t + 1, V of tile t} with LAG, the two that one pipelined iteration of the forward kernel reads,
// {K, V of tile t} without.  A set is always 2 N loads per wave, so that the kernels can wait by count: past the
// end of the walk the last tile's address is asked for again (into a slot nobody reads), and with LAG V of the
// first tile before its start.
template <int D, int BK, int NW, bool BLK, bool LAG>   // BLK: block-wise sparse mask
struct KvStream {
  using Stager = DirectStager<D, BK, NW>;
  static constexpr int N = Stager::N, LOADS = 2 * N;   // per wave: one tile, one set
  Stager stage_k, stage_v;
  int left, k0;           // cursor: tiles left in the run (with a block mask 1; 0: the walk is over), first key row of its tile
  int v0;                 // LAG: first key row of the tile whose V comes with the next set
  int sk;
  OpenTiles open;         // with a block mask, and the end of the run in tiles
  int run_end;
  const char *k_tile, *v_tile, *v_prev;
  int64_t k_step, v_step; // bytes per tile

  __device__ __forceinline__ void init(const MaskDev& mk, const TensorDev& k, const TensorDev& v, int b, int hk, int sk_,
                                       int q_lo, int q_hi, int wave, int lane, const uint8_t* open_flags) {
    sk = sk_;
    TileRun run = visible_tiles<false, BK>(mk, q_lo, q_hi, sk);
    run.start = __builtin_amdgcn_readfirstlane(run.start);   // (results of divisions: keeps what follows scalar)
    left = __builtin_amdgcn_readfirstlane(run.len);
    if (BLK) {
      open.flags = open_flags;
      run_end = run.start + left;
      if (left > 0) {
        open.start(run.start);
        const int tile = open.next(run_end);
        left = tile >= 0;
        run.start = max(tile, 0);
      }
      left = __builtin_amdgcn_readfirstlane(left);
    }
    k0 = run.start * BK;
    k_step = 2 * BK * k.ss;
    v_step = 2 * BK * v.ss;
    k_tile = reinterpret_cast<const char*>((const __bf16*)k.ptr + b * k.sb + hk * k.sh) + run.start * k_step;
    v_tile = reinterpret_cast<const char*>((const __bf16*)v.ptr + b * v.sb + hk * v.sh) + run.start * v_step;
    stage_k.init(k.ss, wave, lane);
    stage_v.init(v.ss, wave, lane);
    v_prev = v_tile;
    v0 = k0;
  }
  __device__ __forceinline__ bool valid() const { return left > 0; }
  // Before the loads of a set: a tile that reaches past the last row is read with clamped row indices
  __device__ __forceinline__ void begin(int wave, int lane) {
    if (k0 + BK > sk) {
      stage_k.clamp(k_step / (2 * BK), sk - k0, wave, lane);
      const int v_row = LAG ? v0 : k0;
      if (v_row + BK > sk) stage_v.clamp(v_step / (2 * BK), sk - v_row, wave, lane);
    }
  }
  __device__ __forceinline__ void load_k(int i, uint32_t lds, int wave) const { stage_k.load_one(k_tile, i, lds, wave); }
  __device__ __forceinline__ void load_v(int i, uint32_t lds, int wave) const { stage_v.load_one(LAG ? v_prev : v_tile, i, lds, wave); }
  // First key row of the cursor's tile, -1 when the walk is over
  __device__ __forceinline__ int cursor() const { return k0 | negative_mask(left - 1); }
  // After them: the cursor moves to the next tile (and stays on the last one when there is none), in PARTS pieces
  // of a few scalar instructions that fit between the matrix instructions of a stream.
  static constexpr int PARTS = 3;
  int move;               // mask: the cursor moves; with a block mask, the number of tiles
  __device__ __forceinline__ void end(int part) {
    if (part == 0) {
      if (LAG) {
        v_prev = v_tile;
        v0 = k0;
      }
      if (!BLK) {
        move = negative_mask(1 - left);
        left += negative_mask(-left);
        k0 += BK & move;
      } else {
        move = 0;
        if (left > 0) {
          const int tile = open.next(run_end);
          left = tile >= 0;
          if (left) move = tile - k0 / BK;
        }
        move = __builtin_amdgcn_readfirstlane(move);
        left = __builtin_amdgcn_readfirstlane(left);
        k0 += move * BK;
      }
      if (LAG) pin(v_prev, v0);
      pin(left, k0);
    }
    if (part == 1) {
      k_tile += BLK ? move * k_step : k_step & (int64_t)move;
      pin(k_tile);
    }
    if (part == 2) {
      v_tile += BLK ? move * v_step : v_step & (int64_t)move;
      pin(v_tile);
    }
  }
  __device__ __forceinline__ void end() {
#pragma unroll
    for (int i = 0; i < PARTS; ++i) end(i);
  }
  // n tiles on; past the end the walk is over
  __device__ __forceinline__ void skip(int n) {
    static_assert(!LAG, "moves K and V of one tile");
    if (BLK) {
      for (int i = 0; i < n; ++i) end();
      return;
    }
    const int more = negative_mask(n - left), m = n & more;
    left = (left - n) & more;
    k0 += m * BK;
    k_tile += m * k_step;
    v_tile += m * v_step;
    pin(left, k0, k_tile, v_tile);
  }
  __device__ __forceinline__ void issue(uint32_t k_lds, uint32_t v_lds, int wave, int lane) {
    begin(wave, lane);
#pragma unroll
    for (int i = 0; i < N; ++i) load_v(i, v_lds, wave);
#pragma unroll
    for (int i = 0; i < N; ++i) load_k(i, k_lds, wave);
    end();
  }
};

// Walk of a key block over (query head of its group, query tile of BQ rows that can see it): per tile the Q and dO
// rows, which all NW waves bring together, and BQ values of the row vector that the wave itself reads (64 lanes: its
// own copy).  A tile is always 2 N + 1 loads per wave; past the end of the walk the last tile is asked for again.
template <int D, int BQ, int NW, bool BLK>   // BLK: block-wise sparse mask
struct QStream {
  using Stager = DirectStager<D, BQ, NW>;
  static constexpr int N = Stager::N, LOADS = 2 * N + 1;
  static_assert(BQ == 64, "a row vector value per lane");
  Stager stage_q, stage_o;
  uint32_t row_off;
  int left, heads, q0;    // cursor: tiles left of this head, heads left (0: the walk is over), first row of its tile
  int run_start, run_len, sq;
  int clamped;            // mask
  OpenTiles open;         // with a block mask
  const char *q_tile, *o_tile, *row_tile;
  int64_t q_step, o_step;                   // bytes per tile
  int64_t q_next, o_next, row_next;         // from the last tile of a head to the first one of the next, bytes

  __device__ __forceinline__ void init(const TensorDev& q, const TensorDev& d_o, const RowvecDev& vec, int b, int hq, int group,
                                       TileRun run, int sq_, int wave, int lane, const uint8_t* open_flags) {
    sq = sq_;
    run_start = __builtin_amdgcn_readfirstlane(run.start);   // (results of divisions: keeps what follows scalar)
    run_len = __builtin_amdgcn_readfirstlane(run.len);
    heads = run_len > 0 ? group : 0;
    left = run_len;
    q0 = run_start * BQ;
    q_step = 2 * BQ * q.ss;
    o_step = 2 * BQ * d_o.ss;
    q_next = 2 * q.sh - (run_len - 1) * q_step;
    o_next = 2 * d_o.sh - (run_len - 1) * o_step;
    row_next = 4 * vec.sh - (run_len - 1) * (int64_t)(4 * BQ);
    q_tile = reinterpret_cast<const char*>((const __bf16*)q.ptr + b * q.sb + hq * q.sh) + run_start * q_step;
    o_tile = reinterpret_cast<const char*>((const __bf16*)d_o.ptr + b * d_o.sb + hq * d_o.sh) + run_start * o_step;
    row_tile = reinterpret_cast<const char*>(vec.ptr + b * vec.sb + hq * vec.sh + q0);
    offsets(BQ, wave, lane);
    clamped = 0;
    if (BLK) {
      open.flags = open_flags;
      if (heads > 0) {
        open.start(run_start);
        const int first = open.next(run_start + run_len);
        if (first >= 0) to_tile(first);
        else heads = 0;
      }
      heads = __builtin_amdgcn_readfirstlane(heads);
    }
  }
  __device__ __forceinline__ void offsets(int valid, int wave, int lane) {
    stage_q.clamp(q_step / (2 * BQ), valid, wave, lane);
    stage_o.clamp(o_step / (2 * BQ), valid, wave, lane);
    row_off = 4 * min(lane, valid - 1);
  }
  __device__ __forceinline__ bool valid() const { return heads > 0; }
  // First row of the cursor's tile, -1 when the walk is over
  __device__ __forceinline__ int cursor() const { return q0 | negative_mask(heads - 1); }
  // To another tile of the cursor's head
  __device__ __forceinline__ void to_tile(int tile) {
    const int n = __builtin_amdgcn_readfirstlane(tile - q0 / BQ);
    q0 += n * BQ;
    q_tile += n * q_step;
    o_tile += n * o_step;
    row_tile += n * 4 * BQ;
  }
  // To the next tile; at the end of the walk the cursor stays where it is.  Without a block mask in PARTS pieces of a few
  // scalar instructions that fit between the matrix instructions of a stream, as in KvStream.
  static constexpr int PARTS = 4;
  int to_next, to_head;   // masks: the cursor moves on in its head, to the next head
  __device__ __forceinline__ void end(int part) {
    if (part == 0) {
      const int not_over = negative_mask(-heads);
      to_next = negative_mask(1 - left);
      to_head = ~to_next & negative_mask(1 - heads);
      heads += ~to_next & not_over;
      left += (run_len & to_head) + not_over;        // (over: the last tile of the last head, for good)
      q0 += (BQ & to_next) - ((run_len - 1) * BQ & to_head);
      pin(heads, left, q0);
    }
    if (part == 1) {
      q_tile += (q_step & (int64_t)to_next) + (q_next & (int64_t)to_head);
      pin(q_tile);
    }
    if (part == 2) {
      o_tile += (o_step & (int64_t)to_next) + (o_next & (int64_t)to_head);
      pin(o_tile);
    }
    if (part == 3) {
      row_tile += ((4 * BQ) & to_next) + (row_next & (int64_t)to_head);
      pin(row_tile);
    }
  }
  __device__ __forceinline__ void advance() {
    if (!BLK) {
#pragma unroll
      for (int i = 0; i < PARTS; ++i) end(i);
      return;
    }
    if (heads == 0) return;
    int tile = open.next(run_start + run_len);
    if (tile < 0) {   // the same tiles of the next head
      if (heads == 1) {
        heads = 0;
        return;
      }
      --heads;
      to_tile(run_start + run_len - 1);
      q0 -= (run_len - 1) * BQ;
      q_tile += q_next;
      o_tile += o_next;
      row_tile += row_next;
      open.start(run_start);
      tile = open.next(run_start + run_len);
    }
    to_tile(tile);
  }
  // Before the loads of a tile: rows past the last one are read as copies of it
  __device__ __forceinline__ void begin(int wave, int lane) {
    const int ragged = negative_mask(sq - BQ - q0);
    if (ragged != clamped) {
      offsets(min(sq - q0, BQ), wave, lane);
      clamped = ragged;
    }
  }
  // Load i of a tile
  __device__ __forceinline__ void load(int i, uint32_t q_lds, uint32_t o_lds, uint32_t row_lds, int wave) const {
    if (i < N) stage_q.load_one(q_tile, i, q_lds, wave);
    else if (i < 2 * N) stage_o.load_one(o_tile, i - N, o_lds, wave);
    else load_dword_to_lds(row_tile, row_off, row_lds);
  }
};

// Products with one hook per LDS operand (NB MFMAs): hook(i) holds independent vector work that goes behind
// them, and the scheduling fence after it keeps it there.  Operands are fetched AHEAD of their use; the first
// AHEAD ones may have been fetched by the caller (`first`).
//   acc[mb][nb] = init[mb] + rows(tile)[row0 + 16 mb ..] * b[ks][nb], operand i = ks * MB + mb
template <int D, int MB, int AHEAD>
__device__ __forceinline__ void rows_fetch(uint32_t tile, const OperandAddr<D>& ad, int row0, bf16x8 (&first)[AHEAD]) {
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) first[i] = rows_operand<D>(tile, ad, row0 + 16 * (i % MB), i / MB);
}
template <int D, int MB, int NB, int AHEAD>
__device__ __forceinline__ void rows_product(uint32_t tile, const OperandAddr<D>& ad, int row0, const bf16x8 (&b)[D / 32][NB],
                                             f32x4 (&acc)[MB][NB], const f32x4 (&init)[MB], const bf16x8 (&first)[AHEAD]) {
  constexpr int N = D / 32 * MB;
  static_assert(AHEAD <= N, "more operands fetched ahead than the product has");
  bf16x8 a[N];
  MatrixPhase prio;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) a[i] = first[i];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + AHEAD < N) a[i + AHEAD] = rows_operand<D>(tile, ad, row0 + 16 * ((i + AHEAD) % MB), (i + AHEAD) / MB);
    const int ks = i / MB, mb = i % MB;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma16(a[i], b[ks][nb], ks == 0 ? init[mb] : acc[mb][nb]);
    __builtin_amdgcn_sched_barrier(0);
  }
}
//   acc[db][nb] += cols(tile)[db, 32-row chunk c] * b[c][nb], operand i = c * (D / 16) + db; b[c] is read when its
//   MFMAs are issued, so a hook may still complete it for a later chunk.
template <int D, int AHEAD>
__device__ __forceinline__ void cols_fetch(uint32_t tile, const OperandAddr<D>& ad, int row0, bf16x8 (&first)[AHEAD]) {
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) first[i] = cols_operand<D>(tile, ad, row0 + 32 * (i / (D / 16)), i % (D / 16));
}
template <int D, int NC, int NB, int AHEAD, class Hook = NoHook>
__device__ __forceinline__ void cols_product(uint32_t tile, const OperandAddr<D>& ad, int row0, const bf16x8 (&b)[NC][NB],
                                             f32x4 (&acc)[D / 16][NB], const bf16x8 (&first)[AHEAD], Hook&& hook = Hook()) {
  constexpr int DB = D / 16, N = NC * DB;
  static_assert(AHEAD <= N, "more operands fetched ahead than the product has");
  bf16x8 a[N];
  MatrixPhase prio;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) a[i] = first[i];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + AHEAD < N) a[i + AHEAD] = cols_operand<D>(tile, ad, row0 + 32 * ((i + AHEAD) / DB), (i + AHEAD) % DB);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[i % DB][nb] = mfma16(a[i], b[i / DB][nb], acc[i % DB][nb]);
    hook(i);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Two row-wise products of the same rows of two tiles, one after the other: acc0 = rows(tile0) * b0, then
// acc1 = rows(tile1) * b1, both from zero.  The first AHEAD operands come fetched.
template <int D, int MB, int NB, int AHEAD>
__device__ __forceinline__ void rows_product_pair(uint32_t tile0, uint32_t tile1, const OperandAddr<D>& ad,
                                                  const bf16x8 (&b0)[D / 32][NB], const bf16x8 (&b1)[D / 32][NB],
                                                  f32x4 (&acc0)[MB][NB], f32x4 (&acc1)[MB][NB],
                                                  const bf16x8 (&first)[AHEAD]) {
  constexpr int N1 = D / 32 * MB, N = 2 * N1;
  bf16x8 a[N];
  MatrixPhase prio;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) a[i] = first[i];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int f = i + AHEAD, f1 = f - N1, i1 = i - N1;
    if (f < N1) a[f] = rows_operand<D>(tile0, ad, 16 * (f % MB), f / MB);
    else if (f < N) a[f] = rows_operand<D>(tile1, ad, 16 * (f1 % MB), f1 / MB);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      if (i < N1) acc0[i % MB][nb] = mfma16(a[i], b0[i / MB][nb], i < MB ? zero : acc0[i % MB][nb]);
      else acc1[i1 % MB][nb] = mfma16(a[i], b1[i1 / MB][nb], i1 < MB ? zero : acc1[i1 % MB][nb]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// One stream of both: s = rows(kt) * q from zero, then o += cols(vt) * p, hook(i) behind operand i of the two.  The
// first operands of the row-wise product come fetched, those of the second are fetched while the first runs.  s has to be the first
// of the two: the forward kernel's max3 reads it in assembly statements, for which the compiler does not wait (common.hpp).
template <int D, int MB, int NB, int AHEAD, class Hook = NoHook>
__device__ __forceinline__ void rows_cols_stream(uint32_t kt, uint32_t vt, const OperandAddr<D>& ad, const bf16x8 (&q)[D / 32][NB],
                                                 f32x4 (&s)[MB][NB], const bf16x8 (&p)[MB / 2][NB], f32x4 (&o)[D / 16][NB],
                                                 const bf16x8 (&first)[AHEAD], Hook&& hook = Hook()) {
  constexpr int DB = D / 16, N1 = D / 32 * MB, N = N1 + MB / 2 * DB;
  static_assert((N - N1) * NB >= 4, "the last of s is in its registers when the stream ends (16 wait states: mfma_results)");
  bf16x8 a[N];
  MatrixPhase prio;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) a[i] = first[i];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int f = i + AHEAD, fc = f - N1, ic = i - N1;
    if (f < N1) a[f] = rows_operand<D>(kt, ad, 16 * (f % MB), f / MB);
    else if (f < N) a[f] = cols_operand<D>(vt, ad, 32 * (fc / DB), fc % DB);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if (i < N1) s[i % MB][nb] = mfma16(a[i], q[i / MB][nb], i < MB ? f32x4{0.f, 0.f, 0.f, 0.f} : s[i % MB][nb]);
      else o[ic % DB][nb] = mfma16(a[i], p[ic / DB][nb], o[ic % DB][nb]);
    }
    hook(i);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Per-element mask of two accumulator tiles, rows base_row .. base_row + 31 (wave-uniform): the lane keeps the entries of
// rows [lo, hi); the others become -inf.  Compares with constants and selects only.
__device__ __forceinline__ void mask_rows32(f32x4& s0, f32x4& s1, int base_row, int g, int lo, int hi, bool check_lo) {
  const int h = hi - base_row - 4 * g, l = lo - base_row - 4 * g;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      f32x4& s = a == 0 ? s0 : s1;
      s[v] = 16 * a + v < h ? s[v] : -INFINITY;
    }
  if (check_lo) {   // wave-uniform
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f32x4& s = a == 0 ? s0 : s1;
        s[v] = 16 * a + v >= l ? s[v] : -INFINITY;
      }
  }
}

}  // namespace burst
