// Shared device-side building blocks of libburstattn's gfx950 kernels: types, the mask, tiles, work-group mapping.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#ifndef BURST_MFMA_PRIO
#define BURST_MFMA_PRIO 2
#endif

namespace burst {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

enum TileClass : int { TILE_SKIP = 0, TILE_FULL = 1, TILE_PARTIAL = 2 };

// Device copy of the visibility description; positions fit in int32 (checked on the host).
// Each axis (query rows, key rows) is a chunk of nseg pieces of seg_len rows; piece s starts at position
// pos0 + s * period and its rows are pos_stride apart.  The pieces are in increasing position order and do
// not overlap (period > (seg_len - 1) * pos_stride, checked on the host), so the position is a strictly
// increasing function of the local row: every "rows whose position is below x" set is a prefix of the chunk,
// and everything the tile logic needs follows from counting such prefixes (rows_lt).
struct MaskDev {
  int32_t causal;
  int32_t q_nseg, k_nseg;
  int32_t q_seg_len, k_seg_len;
  int32_t q_pos0, k_pos0;
  int32_t q_period, k_period;   // 0 with a single piece
  int32_t pos_stride;
  int32_t window;   // causal only: pos(q) - pos(k) < window as well; kNoWindow = unlimited
  // Block-wise sparse mask over local rows (nullptr: none): byte [q_row / blk_q][k_row / blk_k],
  // row pitch blk_pitch bytes, nonzero = the block pair is open.  blk_q is a multiple of 256 and
  // blk_k of 128 (checked on the host), so every tile of every kernel lies inside one block pair.
  const uint8_t* blk;
  int32_t blk_q, blk_k, blk_pitch;
};
constexpr int kMaxBlockCacheTiles = 4096;   // tiles of the walked axis whose open flags fit the LDS cache

// Open flags of the tiles of one axis against a fixed block of the other, cached in LDS once per
// work-group: flags[t] for tile t of TILE rows.  fixed_row: any row of the fixed block.
template <bool WALK_KEYS, int TILE>
__device__ __forceinline__ void fill_open_flags(const MaskDev& mk, uint8_t* flags, int fixed_row, int rows, int tid, int nthreads) {
  const int n = (rows + TILE - 1) / TILE;
  for (int t = tid; t < n; t += nthreads) {
    const int q_blk = WALK_KEYS ? fixed_row / mk.blk_q : (t * TILE) / mk.blk_q;
    const int k_blk = WALK_KEYS ? (t * TILE) / mk.blk_k : fixed_row / mk.blk_k;
    flags[t] = mk.blk[(int64_t)q_blk * mk.blk_pitch + k_blk];
  }
}
constexpr int32_t kNoWindow = 0x7fffffff;   // no position difference reaches it (positions < 2^31 - 1)

// A [batch, seq, heads, D] tensor; strides in elements.
struct TensorDev {
  void* ptr;
  int64_t sb, ss, sh;
  int32_t is_f32;
};
struct RowvecDev {
  float* ptr;
  int64_t sb, sh;
};

// One axis of the mask.
struct AxisMap {
  int32_t nseg, seg_len, pos0, period, stride;
};
template <bool Q_AXIS>
__host__ __device__ __forceinline__ AxisMap axis_of(const MaskDev& mk) {
  return Q_AXIS ? AxisMap{mk.q_nseg, mk.q_seg_len, mk.q_pos0, mk.q_period, mk.pos_stride}
                : AxisMap{mk.k_nseg, mk.k_seg_len, mk.k_pos0, mk.k_period, mk.pos_stride};
}

// Position of local row `row` (rows past the end of the chunk continue the last piece).
__host__ __device__ __forceinline__ int axis_position(const AxisMap& ax, int row) {
  if (ax.nseg <= 1) return ax.pos0 + row * ax.stride;
  int s = row / ax.seg_len;
  s = s < ax.nseg - 1 ? s : ax.nseg - 1;
  return ax.pos0 + s * ax.period + (row - s * ax.seg_len) * ax.stride;
}

// Number of rows r in [0, rows) whose position is below x (x may carry a window: 64-bit).  The
// divisions run on values clipped to the chunk's position span, which fits 32 bits.
__host__ __device__ __forceinline__ int rows_lt(const AxisMap& ax, long long x, int rows) {
  const long long t = x - ax.pos0;
  if (t <= 0 || rows <= 0) return 0;
  const long long span = (long long)(ax.nseg - 1) * ax.period + (long long)(ax.seg_len - 1) * ax.stride;   // position of the last row - pos0
  if (ax.nseg <= 1) {
    if (t > (long long)(rows - 1) * ax.stride) return rows;
    return (int)(((uint32_t)t + (uint32_t)ax.stride - 1u) / (uint32_t)ax.stride);
  }
  if (t > span) return rows;
  uint32_t p = ((uint32_t)t - 1u) / (uint32_t)ax.period;          // last piece that starts below x
  p = p < (uint32_t)(ax.nseg - 1) ? p : (uint32_t)(ax.nseg - 1);
  const uint32_t rem = (uint32_t)t - p * (uint32_t)ax.period;      // > 0
  uint32_t n = (rem + (uint32_t)ax.stride - 1u) / (uint32_t)ax.stride;
  n = n < (uint32_t)ax.seg_len ? n : (uint32_t)ax.seg_len;
  const int tot = (int)(p * (uint32_t)ax.seg_len + n);
  return tot < rows ? tot : rows;
}

// min / max position over local rows [row0, row1), row1 > row0: positions grow with the row
template <bool Q_AXIS>
__host__ __device__ __forceinline__ void range_minmax(const MaskDev& mk, int row0, int row1, int& lo, int& hi) {
  const AxisMap ax = axis_of<Q_AXIS>(mk);
  lo = axis_position(ax, row0);
  hi = axis_position(ax, row1 - 1);
}

// Class of a block whose query positions span [qlo, qhi] and key positions [klo, khi] under a causal
// mask, from the bounding ranges alone (a mixed verdict is always safe).
__host__ __device__ __forceinline__ int classify_ranges(const MaskDev& mk, int qlo, int qhi, int klo, int khi, bool ragged) {
  if (qhi < klo) return TILE_SKIP;                                   // every key lies after every query
  if ((long long)qlo - khi >= mk.window) return TILE_SKIP;           // every key has left every query's window
  if (qlo >= khi && (long long)qhi - klo < mk.window && !ragged) return TILE_FULL;
  return TILE_PARTIAL;
}

// Classify the block of query rows [q0, q1) against key rows [k0, k1) (both already clipped to the
// chunk).  PARTIAL = needs the per-element predicate: the mask edge crosses the block, or the caller
// says so because the register tile also covers rows beyond the end of a chunk.
__host__ __device__ __forceinline__ int classify(const MaskDev& mk, int q0, int q1, int k0, int k1, bool ragged) {
  if (k1 <= k0 || q1 <= q0) return TILE_SKIP;
  if (!mk.causal) return ragged ? TILE_PARTIAL : TILE_FULL;
  int qlo, qhi, klo, khi;
  range_minmax<true>(mk, q0, q1, qlo, qhi);
  range_minmax<false>(mk, k0, k1, klo, khi);
  return classify_ranges(mk, qlo, qhi, klo, khi, ragged);
}

// Row intervals of one axis against ONE fixed position range [olo, ohi] of the other axis: the rows
// that see / are seen by SOME row of the other side are [some_lo, some_hi), those that see / are seen
// by ALL of them [all_lo, all_hi) (possibly empty).  Positions grow with the row, so each set is one
// interval of rows, whatever the number of pieces.
struct RowIntervals {
  int32_t some_lo, some_hi, all_lo, all_hi;
};
template <bool Q_AXIS>
__host__ __device__ __forceinline__ RowIntervals row_intervals(const MaskDev& mk, int olo, int ohi, int rows, bool other_empty) {
  RowIntervals iv{0, 0, 0, 0};
  if (other_empty || rows <= 0) return iv;   // nothing on the other side: every block is empty
  if (!mk.causal) {
    iv.some_hi = iv.all_hi = rows;
    return iv;
  }
  const AxisMap ax = axis_of<Q_AXIS>(mk);
  const long long w = mk.window;
  if (Q_AXIS) {
    // query position p sees key position k iff k <= p < k + window; keys span [olo, ohi]
    iv.some_lo = rows_lt(ax, olo, rows);                    // first p >= olo
    iv.some_hi = rows_lt(ax, (long long)ohi + w, rows);     // first p >= ohi + window
    iv.all_lo = rows_lt(ax, ohi, rows);                     // first p >= ohi
    iv.all_hi = rows_lt(ax, (long long)olo + w, rows);      // first p >= olo + window
  } else {
    // key position k is seen from query position p iff p - window < k <= p; queries span [olo, ohi]
    iv.some_lo = rows_lt(ax, (long long)olo - w + 1, rows);   // first k > olo - window
    iv.some_hi = rows_lt(ax, (long long)ohi + 1, rows);       // end of k <= ohi
    iv.all_lo = rows_lt(ax, (long long)ohi - w + 1, rows);    // first k > ohi - window
    iv.all_hi = rows_lt(ax, (long long)olo + 1, rows);        // end of k <= olo
  }
  return iv;
}

// Class of a tile of `bk` rows against a wave's own rows of the other axis, from its first row: nothing visible,
// all of it visible, or mixed (the per-element mask decides).
struct TileRanges {
  int some_lo, full_lo;
  uint32_t some_len, full_len, end;
  __host__ __device__ __forceinline__ void init(const RowIntervals& iv, int rows, int bk) {
    some_lo = iv.some_lo - bk + 1;
    // (nothing at or behind the last row; an interval that is empty between two rows makes their tile "some", as the
    // ranges of classify() do: a window can fall between the positions of a stride)
    some_len = iv.some_lo < rows ? iv.some_hi - some_lo : 0;
    end = iv.some_hi;
    full_lo = iv.all_lo;
    full_len = max(min(iv.all_hi, rows) - bk + 1 - full_lo, 0);
  }
  __host__ __device__ __forceinline__ bool some(int row0) const { return (uint32_t)(row0 - some_lo) < some_len; }
  __host__ __device__ __forceinline__ bool full(int row0) const { return (uint32_t)(row0 - full_lo) < full_len; }
  // Behind the last tile of which something is visible; so is -1, the end of a walk
  __host__ __device__ __forceinline__ bool behind(int row0) const { return (uint32_t)row0 >= end; }
};

// Rows of one axis that a row of the OTHER axis at position `pos` sees / is seen by: [lo, hi), one interval because
// positions grow with the row.  Per lane, once per work-group; free of divisions for at most two pieces of stride 1.
template <bool KEYS>   // KEYS: the key rows a query sees; else the query rows that see a key
__host__ __device__ __forceinline__ void visible_rows(const MaskDev& mk, int pos, int rows, int& lo, int& hi) {
  lo = 0;
  hi = rows;
  if (!mk.causal) return;
  const AxisMap ax = axis_of<!KEYS>(mk);
  auto below = [&](int x) {   // rows whose position is below x
    const int t = max(x, 0) - ax.pos0;
    if (ax.stride == 1 && ax.nseg <= 2) {
      const int in_first = min(max(t, 0), ax.seg_len), in_second = ax.nseg == 2 ? min(max(t - ax.period, 0), ax.seg_len) : 0;
      return ax.nseg == 2 ? in_first + in_second : min(max(t, 0), rows);
    }
    return rows_lt(ax, (long long)t + ax.pos0, rows);
  };
  if (KEYS) {
    hi = below(pos + 1);                                            // k <= p
    if (mk.window != kNoWindow) lo = below(pos - mk.window + 1);    // k > p - window
  } else {
    lo = below(pos);                                                                  // p >= k
    if (mk.window != kNoWindow && pos <= 0x7fffffff - mk.window) hi = below(pos + mk.window);   // p < k + window
  }
}

// Largest of three (a NaN among them is left out, as by fmaxf).  fmaxf is not folded into it: each of its arguments that the
// compiler cannot prove to be a quiet number costs an instruction that makes it one.  The compiler does not keep an
// assembly statement away from an MFMA whose result it reads: mfma_results() goes before one that may follow closely, or other
// MFMAs stand between (rows_cols_stream).
__device__ __forceinline__ float max3(float a, float b, float c) {
  float m;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(c));
  return m;
}

// Sixteen wait states: the results of the MFMAs before are in their registers.
__device__ __forceinline__ void mfma_results() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15");
  __builtin_amdgcn_sched_barrier(0);
}

// Wait for every outstanding global load of this wave.  Used once, before a tile loop, after the
// loop-invariant register operands were fetched: without it the compiler cannot prove on every
// path that they have landed and re-inserts vmcnt waits inside the loop, which then also wait for
// the tile prefetch issued just before them.
__device__ __forceinline__ void wait_global_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// The tiles of an axis that have any visible pair against the WHOLE other chunk, as up to two runs of
// consecutive tile indices (found by the host; with more runs every tile is launched).  Only these are
// launched: an empty work-group costs a dispatch slot, and many of them in a row starve the other CUs.
struct TileRuns {
  int32_t start[2], len[2];
  __host__ __device__ int total() const { return len[0] + len[1]; }
  __host__ __device__ int tile_of(int i) const { return i < len[0] ? start[0] + i : start[1] + (i - len[0]); }
};

// Tiles of TILE rows along the query axis (Q_AXIS) or the key axis that can hold a pair visible to
// the other side, whose positions span [olo, ohi]: the rows that see / are seen by some row of the other
// side are one interval of rows (row_intervals), hence one run of consecutive tiles.  A tile in the run
// may still turn out empty for a narrower row range; a tile outside it never holds a visible pair.
struct TileRun {
  int32_t start, len;
};
template <bool Q_AXIS, int TILE>
__host__ __device__ __forceinline__ TileRun visible_tiles(const MaskDev& mk, int olo, int ohi, int rows) {
  const RowIntervals iv = row_intervals<Q_AXIS>(mk, olo, ohi, rows, false);
  if (iv.some_lo >= iv.some_hi) return TileRun{0, 0};
  const int first = iv.some_lo / TILE;
  return TileRun{first, (iv.some_hi + TILE - 1) / TILE - first};
}

// Scope of a stream of MFMAs: the wave runs at raised issue priority.  A SIMD issues one vector-class
// instruction at a time and picks the oldest ready wave; without this, a co-resident wave in a
// dense vector phase (softmax, dS) keeps winning the issue slot and the matrix pipe idles, although
// an MFMA of 16 clocks needs only one slot in four.
struct MatrixPhase {
  __device__ __forceinline__ MatrixPhase() { __builtin_amdgcn_s_setprio(BURST_MFMA_PRIO); }
  __device__ __forceinline__ ~MatrixPhase() { __builtin_amdgcn_s_setprio(0); }
};

struct NoHook {
  __device__ __forceinline__ void operator()(int) const {}
};

// Work-group index -> (kv key = batch*Hkv + kv head, head within group, tile).  Work-group n runs on XCD
// n mod 8 (they are dealt round-robin), each XCD with its own L2.
//  - Keys that fill whole rounds of eight go one to an XCD, so its K/V (or Q/dO) stream is shared in that L2.
//  - The remaining n_keys mod 8 keys are dealt tile by tile over all XCDs (with one XCD per key, 16/2 heads
//    kept two XCDs busy and six idle: a forward step of 8192 rows took 1058 us, now 294; dQ 1331, now 365).
//    They come first, so that the launch ends on the light tiles of the other keys.
// Heavier tiles start first: under a causal mask a query tile is heavier the higher its rows (HIGH_FIRST), a
// key tile the lower its rows.  That is also what keeps the work-groups that share an L2 in step: the ones
// running together then walk the other axis at the same place at the same time, so each tile of it is fetched
// from HBM once.  The heads of a group take the same tile one after the other.  A launch of few work-groups per CU
// (kShortLaunch) whose walks are uneven runs the keys of an XCD side by side, heaviest tiles of all of them first,
// because there the balance of the last round counts more than the L2 share; where all walks are alike there is nothing
// to balance, and as many streams as keys go through an L2 for nothing.  32 heads, d = 128 (4 keys per XCD), us key by
// key and side by side:
//   own shard, causal: forward 8192 rows (128 work-groups per XCD) 618, 605; 12288 (192) 1061, 1025; 16384 (256) 1827,
//   1835; 18432 (288) 2417, 2376; 32768 (512) 7442, 7520.  dQ 748, 722; 1430, 1415; 2556, 2541; 3235, 3240; 10020,
//   10070.  dK/dV, whose tiles are half as high, 8192 rows (256) 1011, 991; 12288 (384) 2064, 2082; 16384 3616, 3637.
//   an earlier shard of the zigzag split, whose keys every query sees: forward 16384 rows 1782, 1777; dQ 2447, 2455; dK/dV,
//   whose launch is half as long, 8192 rows (128) 942, 955; 12288 (192) 2010, 2089; 16384 (256) 3519, 3911, with
//   0.95 and 2.59 GB of memory traffic (forward 0.67 and 1.48, dQ 0.81 and 1.62).
//   block pattern of density 0.25 over 512-token blocks, 16384 rows, forward and backward of a ring: the keys of
//   its earlier and later shards side by side 21.99 ms, one after the other 22.35.
struct BlockMap {
  int key, head_in_group, tile;
  bool valid;
};
constexpr int kShortLaunch = 256;   // work-groups per XCD (32 CUs)
template <bool HIGH_FIRST>
__host__ __device__ __forceinline__ BlockMap map_block(int n, int n_keys, int group, int tiles, bool side_by_side) {
  const int per_key = group * tiles, full = n_keys >> 3, rest = n_keys & 7;
  const int rest_items = rest * per_key, rest_blocks = (rest_items + 7) & ~7;
  BlockMap m;
  int t;
  if (n < rest_blocks) {
    const int j = n / rest;
    m.key = full * 8 + n - j * rest;
    t = j / group;
    m.head_in_group = j - t * group;
    m.valid = n < rest_items;
  } else {
    const int slot = (n - rest_blocks) >> 3, xcd = n & 7;
    int local_key, in_key;
    if (side_by_side) {
      const int width = full * group;
      t = slot / width;
      const int w = slot - t * width;
      local_key = w / group;
      m.head_in_group = w - local_key * group;
    } else {
      local_key = slot / per_key;
      in_key = slot - local_key * per_key;
      t = in_key / group;
      m.head_in_group = in_key - t * group;
    }
    m.key = local_key * 8 + xcd;
    m.valid = local_key < full;
  }
  m.tile = HIGH_FIRST ? tiles - 1 - t : t;
#ifdef __HIP_DEVICE_COMPILE__   // results of divisions, which the compiler leaves in vector registers
  m.key = __builtin_amdgcn_readfirstlane(m.key);
  m.head_in_group = __builtin_amdgcn_readfirstlane(m.head_in_group);
  m.tile = __builtin_amdgcn_readfirstlane(m.tile);
#endif
  return m;
}
inline bool short_launch(int n_keys, int group, int tiles) { return (n_keys >> 3) * group * tiles <= kShortLaunch; }
inline int mapped_grid(int n_keys, int group, int tiles) {
  const int per_key = group * tiles;
  return (((n_keys & 7) * per_key + 7) & ~7) + (n_keys >> 3) * 8 * per_key;
}

}  // namespace burst
