// Forward step kernel: O_ij, Lse_cur of a query chunk against one key/value chunk (Eq. 5-6),
// optionally folded into the running (O_i, Lse_i) in the epilogue (forward algorithm).
//
// One work-group = 8 waves = 256 query rows of one (batch, head) at d = 128, 4 waves = 128 rows at d = 64; wave w owns rows
// [32w, 32w+32).  The key/value chunk (or several, of consecutive ring steps) streams through LDS in tiles of 64 rows.  Everything is
// computed transposed so that a lane always owns query rows (two of them):
//   S^T = K Q^T   (A = K rows from LDS, B = Q held in registers),
//   P^T = exp2(..) in the accumulator registers, packed to bf16 and fed straight back as the B operand of
//   O^T = V^T P^T (A = V columns via transposing LDS reads).
//
// What bounds it at d = 128, where two waves share a SIMD: the matrix pipe and the vector unit need about the same time for a tile (64 MFMAs of
// 16 clocks; 117 vector instructions, of them 32 exponentials, about 900 clocks for a wave alone), and the chip
// holds a power limit on top.  So the two waves of a SIMD take the phases in turn, and the products use
// 16x16x32 MFMAs, which draw less than 32x32x16 on real data (register-fed, random operands: 2050-2110 against
// 1840-1900 TFLOP/s; with operands that change from MFMA to MFMA 1900-1934 against 1786-1817).
// Tiles arrive by direct global -> LDS loads: no staging registers, no LDS store instructions.
// 131072 x 131072 rows x 32 heads, zigzag: 127.5 -> 109.1 ms (1103 -> 1290 TFLOP/s) on one card.  Counters: matrix pipe 66 % busy
// at 1.86 GHz, where zeros as data run at 2.24 GHz in the same clocks a tile (16384 x 16384 rows: 1727 and 1456 us).
//
// At d = 64 the vector unit is the bound (half the matrix work for the same scores): a tile costs a wave 32 exponentials of 16
// clocks and 85 other vector instructions of 4, and 32 MFMAs take an issue slot of 4 each, 980 clocks a SIMD.  One wave alone, or
// two that take turns, do not issue that fast (a vector instruction every 6 to 9 clocks), three do nearly: a wave needs 158
// registers and a work-group of four 52 KB of LDS, so three work-groups share a CU and fill each other's matrix
// phases, prologues and epilogues without a common rhythm.  Counters: vector unit 81 % busy, matrix pipe 52 % (32 heads x 16384 rows, full); 58 and 34 %
// in a step of 1500 rows, 4 x 12 heads, which does not fill the chip for long enough.  Eight waves in turns, and this, us: 12 heads x 24749 rows 2140, 2050; 32 heads x
// 16384 (an earlier shard) 1153, 1080; 64 x 8548 causal, batch 2, 1390, 1240; with a window (32 heads x 3010, batch 2) 98, 75; one step of 1500
// rows, 4 x 12 heads 67, 47; 1 head x 20000 rows, 157 work-groups 330, 266.  Raised priority of the MFMAs, 2, 3 or 4 operands
// ahead and a fence between the exponentials make no difference here.
//
// A launch of few query tiles is bound by its longest walk, a chain of products and softmax that leaves most CUs idle: there the four
// waves of a work-group share 32 query rows and deal the key tiles among themselves (SPLIT; when: split_walks).
#include "common.hpp"
#include "kernels.hpp"
#include "mfma16.hpp"

namespace burst {

template <int D>
constexpr int kFwdWaves = D == 128 ? 8 : 4;     // two waves per SIMD that take turns; three work-groups per CU
template <int D>
constexpr int kFwdBQ = 32 * kFwdWaves<D>;   // query rows per work-group: 32 per wave
template <int D>
constexpr int kFwdSlots = D == 128 ? 4 : 3;   // tiles of K and V in LDS

// Work-groups whose waves share their query rows (SPLIT)
constexpr int kSplitWaves = 4, kSplitBQ = 32;
struct SplitRow {
  float m, l, lse_before;   // of a wave and a row: maximum and sum of its keys, the running Lse (the first wave's)
};

// The maxima of the rows' scores in the last tiles of a walk, and the rounds each wave has posted them for, in LDS.  A wave that posts
// for round t + 2 knows of every other one that it has posted for round t at least: it does not read tiles before round t - 1 any
// more, and four rounds are kept.  (A wave's LDS instructions complete in order.)
struct SplitPosts {
  static constexpr int ROUNDS = 4, TILES = ROUNDS * kSplitWaves, BYTES = 16 + TILES * kSplitBQ * 4;
  typedef volatile __attribute__((address_space(3))) int* lds_ints;
  typedef volatile __attribute__((address_space(3))) float* lds_floats;
  lds_bytes lds;   // rounds posted: [wave]; maxima: [tile % TILES][row]
  __device__ __forceinline__ lds_ints posted() const { return (lds_ints)lds; }
  __device__ __forceinline__ lds_floats maxima(int tile) const { return (lds_floats)(lds + 16) + (tile & (TILES - 1)) * kSplitBQ; }
  __device__ __forceinline__ void init(int tid) const {
    if (tid < kSplitWaves) posted()[tid] = 0;
  }
  // The rows of nb are 16 nb + lane % 16; the lanes of a row have the same value
  __device__ __forceinline__ void post(int round, int wave, int lane, const float (&top)[2]) const {
    const lds_floats m = maxima(round * kSplitWaves + wave);
    if (lane < 16) {
      m[lane] = top[0];
      m[16 + lane] = top[1];
    }
    keep_order();
    done(round, wave, lane);
  }
  // All of the wave's tiles of rounds up to `round` are there
  __device__ __forceinline__ void done(int round, int wave, int lane) const {
    if (lane == 0) posted()[wave] = round + 1;
    keep_order();
  }
  __device__ __forceinline__ float top(int tile, int nb, int r) const { return maxima(tile)[16 * nb + r]; }
  // read() again and again until the tiles between the wave's last one and this one are there: those of this round of the waves
  // before it, and those of the round before of the waves behind it.
  template <class Read>
  __device__ __forceinline__ void wait(int round, int wave, int lane, Read&& read) const {
    const int w = lane & (kSplitWaves - 1), need = w < wave ? round + 1 : w > wave ? round : 0;
    for (;;) {
      const int have = posted()[w];
      keep_order();
      read();
      if (__all(have >= need)) return;
    }
  }
};

// Largest value of the four lanes r, r + 16, r + 32 and r + 48, without the LDS
__device__ __forceinline__ float max_of_row(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  x = max3(__builtin_bit_cast(float, (uint32_t)a[0]), __builtin_bit_cast(float, (uint32_t)a[1]), -INFINITY);
  const uint32_t v = __builtin_bit_cast(uint32_t, x);
  const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return max3(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]), -INFINITY);
}

// BLK: with a block-wise sparse mask; MULTI: more than one step.  (A single step's arguments are asked for at once at the start;
// steps picked by a variable are a second round trip, 1-2 us of a launch: dK/dV of three steps of 1500 rows 241, 246 us.)
// SPLIT: the waves share 32 query rows and deal the key tiles among themselves.
template <int D, int NW, bool BLK, bool MULTI, bool SPLIT>
__global__ __launch_bounds__(64 * NW, SPLIT ? 2 : D == 128 ? 1 : 3) void step_fwd_kernel(FwdParams p) {
  constexpr int BK = 64, MB = BK / 16, NB = 2, DK = D / 32, DB = D / 16, BQ = SPLIT ? 32 : 32 * NW, NT = 64 * NW;
  constexpr int TILE = BK * 2 * D, SLOTS = SPLIT ? NW : kFwdSlots<D>;
  constexpr int AHEAD = SPLIT && MULTI && D == 128 ? 2 : kAhead16;   // (registers)
  constexpr bool TURNS = D == 128 && !SPLIT;   // the waves of a SIMD take turns
  extern __shared__ __attribute__((aligned(1024))) char smem[];  // [SLOTS][K tile, V tile], SplitRow[NW][BQ] and SplitPosts (SPLIT), open flags

  // (a kernel argument indexed with a variable would be copied to scratch memory: read through the argument pointer)
  typedef const __attribute__((address_space(4))) FwdParams* args_ptr;
  const FwdParams& args = *(const FwdParams*)(args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  const int group = p.q_heads / p.kv_heads;
  const BlockMap bm = map_block<true>(blockIdx.x, p.batch * p.kv_heads, group, p.q_runs.total(), p.q_side_by_side);
  if (!bm.valid) return;
  const int b = __builtin_amdgcn_readfirstlane(bm.key / p.kv_heads), hk = bm.key - b * p.kv_heads, hq = hk * group + bm.head_in_group;

  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: everything derived from it stays wave-uniform
  const int sq = p.sq;
  const int n_steps = MULTI ? p.n_steps : 1;
  const MaskDev q_side = p.step[0].mask;   // all steps have the same
  const int q_blk0 = p.q_runs.tile_of(bm.tile) * BQ;     // first row of the work-group
  const int q_blk1 = min(q_blk0 + BQ, sq);
  const int q_w0 = SPLIT ? q_blk0 : q_blk0 + wave * 32;  // first row of the wave
  const int q_w1 = min(q_w0 + 32, sq);                   // may be <= q_w0: the wave only helps staging

  // Q as the B operand of S^T = K Q^T: lane holds rows q_w0 + 16 nb + r, columns 32 ks + 8g .. +7
  bf16x8 qreg[DK][NB];
  int q_pos[NB], klo[NB], khi[NB];   // positions of the lane's query rows, the key rows they see of a step
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = min(q_w0 + 16 * nb + r, sq - 1);
    q_pos[nb] = axis_position(axis_of<true>(q_side), row);
    const __bf16* src = (const __bf16*)p.q.ptr + b * p.q.sb + hq * p.q.sh + (int64_t)row * p.q.ss + 8 * g;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) qreg[ks][nb] = *reinterpret_cast<const bf16x8*>(src + ks * 32);
  }

  f32x4 o[DB][NB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) o[db][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c = p.scale * kLog2e, slack = kLazyLog2 / c;
  // running maximum, what a score must exceed for a rescale, c * maximum (0 while there is none), running sum
  float m_run[NB] = {-INFINITY, -INFINITY}, limit[NB] = {-INFINITY, -INFINITY}, msub[NB] = {0.f, 0.f};
  f32x4 l_run[NB] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // four independent chains
  float m_top[NB] = {-INFINITY, -INFINITY};   // MULTI: largest maximum of the steps so far
  float m_sums[NB] = {-INFINITY, -INFINITY};   // SPLIT: the maximum that this wave's sums are against
  constexpr int ROWS = SPLIT ? NW * BQ * (int)sizeof(SplitRow) : 0;
  const SplitPosts posts{(lds_bytes)smem + SLOTS * 2 * TILE + ROWS};
  int round = 0;   // SPLIT: of NW tiles, over all steps
  if constexpr (SPLIT) {
    static_assert(NW == kSplitWaves, "waves that post");
    posts.init(tid);
    __syncthreads();
  }

  // Positions of the work-group's and the wave's query rows
  int qlo_blk, qhi_blk, qlo_w = 0, qhi_w = 0;
  range_minmax<true>(q_side, q_blk0, q_blk1, qlo_blk, qhi_blk);
  if (q_w0 < q_w1) range_minmax<true>(q_side, q_w0, q_w1, qlo_w, qhi_w);

  // Open flags of the key tiles against this work-group's query block (block-wise sparse mask)
  uint8_t* open_flags = nullptr;
  if (BLK) {
    open_flags = reinterpret_cast<uint8_t*>(smem + SLOTS * 2 * TILE + ROWS + (SPLIT ? SplitPosts::BYTES : 0));
    fill_open_flags<true, BK>(q_side, open_flags, q_blk0, p.step[0].sk, tid, NT);
    __syncthreads();
  }
  OperandAddr<D> ad;
  ad.init(lane);
  TileRanges tiles;   // class of a step's key tiles against this wave's 32 query rows
  bool windowed;
  uint32_t lds0 = (uint32_t)(uintptr_t)(lds_bytes)smem;

  // A wave's work on a tile is a matrix phase and a vector phase of about the same length, and the two waves of
  // a SIMD take them in turn: while waves 0-3 run iteration t's products, waves 4-7 (one barrier behind) run
  // their softmax, and the other way round.  Iteration t:
  //   matrix phase: S(t+1) = K Q^T and O += V^T P(t), from set t = {K of tile t+1, V of tile t} in slot t mod 4
  //   vector phase: P(t+1) from S(t+1)
  // A barrier ends every phase.  Set t+3 is asked for in the matrix phase of iteration t (its slot held set t-1,
  // which the later half finished a barrier ago).  A wave waits for its share of set t+2 before the barrier that
  // ends its vector phase of iteration t, so that both halves' shares of set t+1 are there before either half's
  // vector phase of iteration t, which ends with the first operand fetches of the next matrix phase.  Iteration -1 has
  // no such barrier before it: the later half waits for its share of set 0 where it drops behind by a barrier.
  // The tiles of which a wave's rows see something are one run of the walk.  Before and behind it the wave only asks for
  // its share of the loads and meets the others: what its rows may not see does not reach them, be it infinite or NaN
  // (zeros in place of P would let 0 * inf through), and in a step of few query rows the waves without rows leave the
  // matrix pipe and the LDS to the others: one query row, 32/8 heads, 4096 keys, d = 128: 94 us with all waves in the
  // products, 70 so (dQ 121 and 82); a 1024-token window 379 and 367.
  // The last iteration forms a product S nobody reads (of a tile it has): a quarter of a tile's time per work-group,
  // where a second copy of the loop's end cost the registers of the operand prefetch (1 % slower).
  // Raised priority of the matrix phase: 3-6 % (16384 rows x 32 heads 1810 and 1910 us, 32768 rows 7100 and 7430); with both
  // at priority 0 the waves' phases disturb each other.  dQ 1-3 %, dK/dV 1-6 %.
  auto k_lds = [&](int s_) { return lds0 + s_ * 2 * TILE; };
  auto v_lds = [&](int s_) { return lds0 + s_ * 2 * TILE + TILE; };
  using Walk = KvStream<D, BK, SPLIT ? 1 : NW, BLK, TURNS>;
  constexpr int LOADS = Walk::LOADS, NL = Walk::N;
  // The steps one after the other; the state stays in registers
#pragma clang loop unroll(disable)
  for (int step = 0; step < n_steps; ++step) {
    const FwdStep& st = MULTI ? args.step[step] : p.step[0];
    const MaskDev mk = st.mask;
    const int sk = st.sk;
    windowed = mk.window != kNoWindow;
    if (step > 0) {   // a step's maximum is its own (see softmax)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) limit[nb] = -INFINITY;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) visible_rows<true>(mk, q_pos[nb], sk, klo[nb], khi[nb]);
    tiles.init(row_intervals<false>(mk, qlo_w, qhi_w, sk, q_w0 >= q_w1), sk, BK);
    Walk walk;
    walk.init(mk, st.k, st.v, b, hk, sk, qlo_blk, qhi_blk, SPLIT ? 0 : wave, lane, open_flags);
    wait_global_loads();
    if (step > 0 && !SPLIT) __syncthreads();   // the later half may still read the last tiles of the step before
    pin(lds0);   // (LDS addresses worked out once for all steps would cost the registers)
    f32x4 s[MB][NB];
    bf16x8 pp[MB / 2][NB];
    // Scores of the tile at key row k0_ without those of pairs that are not visible
    auto mask_scores = [&](int k0_) {
      if (!tiles.full(k0_)) {
#pragma unroll
        for (int half = 0; half < MB / 2; ++half)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) mask_rows32(s[2 * half][nb], s[2 * half + 1][nb], k0_ + 32 * half, g, klo[nb], khi[nb], windowed);
      }
    };
    // Largest score among this lane's keys of the tile (a query row's keys are spread over four lanes)
    auto lane_max = [&](int nb) {
      float m5[5];   // eight v_max3_f32 for sixteen scores (fifteen with fmaxf: 1795 and 1769 us at 16384 rows, 32 heads, d = 128)
#pragma unroll
      for (int i = 0; i < 5; ++i)
        m5[i] = max3(s[3 * i / 4][nb][3 * i % 4], s[(3 * i + 1) / 4][nb][(3 * i + 1) % 4], s[(3 * i + 2) / 4][nb][(3 * i + 2) % 4]);
      return max3(max3(m5[0], m5[1], m5[2]), max3(m5[3], m5[4], s[3][nb][3]), -INFINITY);
    };
    auto row_max = [&](float mx) {
      const float m = fmaxf(mx, __shfl_xor(mx, 16, 64));
      return fmaxf(m, __shfl_xor(m, 32, 64));
    };
    // The running maximum of a row whose keys in a tile reach m_new, where some row of the wave has grown
    auto raise = [&](int nb, float m_new) {
      bool fresh = false;   // the row has seen no key of this step, and sees none in this tile
      if (MULTI) {
        // A row's P at its maximum is one and rounds to bf16 exactly.  A step that kept the maximum of the steps
        // before would lose that: 8 steps of 512 rows, window 700, error of O against 64 bits 1.64e-3 so, 1.17e-3
        // with a maximum for each step.  It is let down to 2^-12 of the largest at most: a step below that weighs little, and
        // fp32 keeps its headroom, sums of P of up to 2^18 a key (with 2^-6 heads scaled by 0.5 to 2 had 1 % more error).
        m_top[nb] = fmaxf(m_top[nb], m_new);
        const bool first = limit[nb] == -INFINITY;
        fresh = first && m_new == -INFINITY;
        m_new = fresh ? m_run[nb] : fmaxf(m_new, first ? m_top[nb] - 2.f * slack : m_run[nb]);
      } else {
        m_new = fmaxf(m_run[nb], m_new);
      }
      m_run[nb] = m_new;
      limit[nb] = fresh ? -INFINITY : m_new + slack;
      msub[nb] = (m_new == -INFINITY) ? 0.f : c * m_new;
    };
    auto grows = [&](const float (&x)[NB]) { return __any(x[0] > limit[0] || x[1] > limit[1]); };
    auto follow = [&](const float (&x)[NB]) {   // a tile of the walk, with the rows' maxima x
      if (!grows(x)) return;
      raise(0, x[0]);
      raise(1, x[1]);
    };
    // The sums so far, of weights against m_old, against m_new
    auto rescale = [&](int nb, float m_old, float m_new) {
      const float alpha = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(c * (m_old - m_new));
      l_run[nb] *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[db][nb][v] *= alpha;
    };
    // P = exp2(c S - c m) as packed bf16; the row sum is taken in fp32 before rounding (Lse must hold to
    // 1e-3 also for rows with a handful of keys).  Eight scores at a time: enough to cover the latency of the
    // exponential, few enough to keep the intermediate values out of the register budget.  The fence keeps the
    // groups apart: with the 32 exponentials in a row the d = 64 kernel is 2-3 % slower (12 heads x 12000 rows 665, 636 us).
    auto exponentials = [&](const float (&offset)[NB]) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int ch = 0; ch < MB / 2; ++ch) {
          f32x4 &x = s[2 * ch][nb], &y = s[2 * ch + 1][nb];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            x[v] = __builtin_amdgcn_exp2f(c * x[v] - offset[nb]);
            y[v] = __builtin_amdgcn_exp2f(c * y[v] - offset[nb]);
          }
          l_run[nb] += x + y;
          pp[ch][nb] = pack_pair(x, y);
          __builtin_amdgcn_sched_barrier(0);
        }
    };
    // P of the tile at key row k0_, of which the wave sees something, from its scores
    auto softmax = [&](int k0_) {
      mask_scores(k0_);
      // Rescale lazily: keep a stale maximum while no row of the wave has grown by more than
      // 2^kLazyLog2 (any common per-row offset gives the same result; fp32 has the headroom).  A row has
      // grown exactly if one of its four lanes has, and the vote runs over the whole wave, so the lanes
      // of a row exchange their maxima only when a rescale happens: the steady state has no cross-lane
      // traffic (the exchange goes through LDS and costs a round trip the wave cannot fill).
      float mx[NB];
      bool grow = false;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        mx[nb] = lane_max(nb);
        grow |= mx[nb] > limit[nb];
      }
      if (__any(grow)) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const float m_old = m_run[nb];
          raise(nb, row_max(mx[nb]));
          rescale(nb, m_old, m_run[nb]);
        }
      }
      exponentials(msub);
    };
    if constexpr (SPLIT) {
      // Round after round, of NW tiles: the wave has tile `wave` of each in a slot of its own; K of the next one comes behind the
      // products of S, V behind O of the tile before.  P is formed against the maximum that one walk over all tiles would have at
      // that tile, so that it rounds to the same bf16 numbers as in the other kernels: the waves post their rows' maxima of every
      // tile, and each follows them tile by tile up to its own.  That needs the tiles before it only, which wait for earlier ones
      // at most: every wait ends.  The products of O, of the tile before, stand between a post and the reading.
      // Against a maximum of its own in each wave O would be 1e-3 from what the other kernels give for the same row.  us so and with
      // posts, d = 128 (d = 64): 4 x 1024 rows 13.8, 14.7 (10.7, 10.7); 1 x 8192 62, 70 (46, 48); causal 1 x 16384 121, 138 (87, 96); four
      // steps of 8 x 2048 79, 90 (45, 51).  With a barrier for each round 1 x 8192 takes 85 (48).
      const uint32_t kt = k_lds(wave), vt = v_lds(wave);
      WaveStager<D, BK, D == 64> k_rows, v_rows;
      k_rows.init(st.k.ss, lane);
      v_rows.init(st.v.ss, lane);
      auto load_k = [&]() { k_rows.load(walk.k_tile, st.k.ss, sk - walk.k0, kt, lane); };
      const int round0 = round, n_tiles = walk.left;   // (rounds are counted over all steps; n_tiles: without a block mask)
      walk.skip(wave);
      if (walk.valid()) {
        load_k();
        bool live = false, more = true;
        bf16x8 first[AHEAD];
        auto add_o = [&]() {   // P V of the tile before
          if (more) wait_loads<NL>();
          else wait_loads<0>();
          if (live) {
            cols_fetch<D, AHEAD>(vt, ad, 0, first);
            cols_product<D, MB / 2, NB, AHEAD>(vt, ad, 0, pp, o, first);
          }
        };
        any_value(pp);
        wait_loads<0>();        // K of the first one
        for (;; ++round) {
          const int kb = walk.k0;
          const char* const v_tile = walk.v_tile;
          walk.skip(NW);
          more = walk.valid();
          const bool now = tiles.some(kb);
          const f32x4 zero[MB] = {};
          float top[NB] = {-INFINITY, -INFINITY};
          if (now) {
            rows_fetch<D, MB, AHEAD>(kt, ad, 0, first);
            rows_product<D, MB, NB, AHEAD>(kt, ad, 0, qreg, s, zero, first);
            mfma_results();
          }
          if (more) load_k();
          if (now) {
            mask_scores(kb);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) top[nb] = max_of_row(lane_max(nb));
          }
          posts.post(round, wave, lane, top);
          add_o();
          v_rows.load(v_tile, st.v.ss, sk - kb, vt, lane);
          live = now;
          float x[NW][NB];   // of the NW tiles up to this one; before the step's first -inf
          posts.wait(round, wave, lane, [&]() {
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
              for (int nb = 0; nb < NB; ++nb) x[i][nb] = posts.top((round - 1) * NW + wave + 1 + i, nb, r);
          });
          float most[NB];
#pragma unroll
          for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
              if (round == round0 && i + wave < NW - 1) x[i][nb] = -INFINITY;
              if (i == NW - 1) most[nb] = max3(max3(x[0][nb], x[1][nb], x[2][nb]), x[3][nb], -INFINITY);
            }
          if (grows(most)) {
#pragma unroll
            for (int i = 0; i < NW; ++i) follow(x[i]);
          }
          if (live) {
            if (__any(m_run[0] != m_sums[0] || m_run[1] != m_sums[1])) {
#pragma unroll
              for (int nb = 0; nb < NB; ++nb) {
                rescale(nb, m_sums[nb], m_run[nb]);
                m_sums[nb] = m_run[nb];
              }
            }
            exponentials(msub);
          }
          if (!more) break;
          wait_loads<NL>();     // K of the next one
        }
        ++round;
        add_o();
      }
      if (MULTI && step + 1 < n_steps) {   // and the tiles behind the wave's last one, for the maximum the next step starts with
        int tile = round > round0 ? (round - 1) * NW + wave + 1 : round0 * NW;
        stores_barrier<0>();
        for (; tile < round0 * NW + n_tiles; ++tile) {
          const float x[NB] = {posts.top(tile, 0, r), posts.top(tile, 1, r)};
          follow(x);
        }
        round = round0 + (n_tiles + NW - 1) / NW;
        posts.done(round - 1, wave, lane);   // (also where the last round had no tile for it)
      }
    } else if (!TURNS) {   // tile t in slot t mod 3: both products and the softmax one after the other, a barrier for each tile
      if (walk.valid()) {
        int kb = walk.cursor();
        walk.issue(k_lds(0), v_lds(0), wave, lane);
        int kc = walk.cursor();
        walk.issue(k_lds(1), v_lds(1), wave, lane);
        int slot = 0;
        do {
          wait_loads_barrier<LOADS>();   // tile t; and all waves have left tile t-1
          const int free_slot = slot == 0 ? 2 : slot - 1;
          const int kn = walk.cursor();
          walk.issue(k_lds(free_slot), v_lds(free_slot), wave, lane);
          if (tiles.some(kb)) {
            const f32x4 zero[MB] = {};
            bf16x8 first[AHEAD];
            rows_fetch<D, MB, AHEAD>(k_lds(slot), ad, 0, first);
            rows_product<D, MB, NB, AHEAD>(k_lds(slot), ad, 0, qreg, s, zero, first);
            cols_fetch<D, AHEAD>(v_lds(slot), ad, 0, first);
            mfma_results();
            softmax(kb);
            cols_product<D, MB / 2, NB, AHEAD>(v_lds(slot), ad, 0, pp, o, first);
          }
          kb = kc;
          kc = kn;
          slot = slot == 2 ? 0 : slot + 1;
          pin(kb, kc, slot);
        } while (kb >= 0);
        wait_global_loads();             // tiles past the end of the walk
      }
    } else if (walk.valid()) {
      int kb = walk.k0;   // iteration t: kb, kc, kd are the first rows of tiles t+1, t+2, t+3
      walk.issue(k_lds(3), v_lds(3), wave, lane);   // set -1
      int kc = walk.cursor();
      walk.issue(k_lds(0), v_lds(0), wave, lane);   // set 0
      int kd = walk.cursor();
      walk.issue(k_lds(1), v_lds(1), wave, lane);   // set 1
      int kn = walk.cursor();
      walk.issue(k_lds(2), v_lds(2), wave, lane);   // set 2
      wait_loads_barrier<3 * LOADS>();              // set -1
      if (wave >= NW / 2) wait_loads_barrier<2 * LOADS>();   // set 0: the first half's first vector phase reads its K
      int slot = 3;
      bool live;
      bf16x8 first[AHEAD];
      any_value(s);
      any_value(pp);
      any_value(first);
      for (;;) {   // iterations -1 .., up to the wave's first tile
        live = tiles.some(kb);
        if (live) {
          const f32x4 zero[MB] = {};
          rows_fetch<D, MB, AHEAD>(k_lds(slot), ad, 0, first);
          rows_product<D, MB, NB, AHEAD>(k_lds(slot), ad, 0, qreg, s, zero, first);
        }
        wait_loads_barrier<2 * LOADS>();            // set 0 (later ones have been waited for)
        slot = (slot + 1) & 3;
        if (live) {
          mfma_results();   // (in the loop below the products of P stand between)
          softmax(kb);
          rows_fetch<D, MB, AHEAD>(k_lds(slot), ad, 0, first);
        }
        wait_loads_barrier<LOADS>();
        kb = kc;
        kc = kd;
        kd = kn;
        if (live || kb < 0) break;
        kn = walk.cursor();
        walk.issue(k_lds((slot + 3) & 3), v_lds((slot + 3) & 3), wave, lane);
      }
      if (live) {
        for (;;) {
          const uint32_t kt = k_lds(slot), vt = v_lds(slot);
          // ---- matrix phase
          kn = walk.cursor();
          walk.begin(wave, lane);
          const int slot3 = (slot + 3) & 3;
          const uint32_t kl = k_lds(slot3), vl = v_lds(slot3);
          rows_cols_stream<D, MB, NB, AHEAD>(kt, vt, ad, qreg, s, pp, o, first, [&](int i) {
            if (i >= 1 && i < 1 + NL) walk.load_v(i - 1, vl, wave);
            if (i >= 1 + NL && i < 1 + 2 * NL) walk.load_k(i - 1 - NL, kl, wave);
            if (i >= 1 + 2 * NL && i < 1 + 2 * NL + walk.PARTS) walk.end(i - 1 - 2 * NL);
          });
          if (tiles.behind(kb)) break;
          phase_barrier();
          // ---- vector phase
          softmax(kb);
          slot = (slot + 1) & 3;
          rows_fetch<D, MB, AHEAD>(k_lds(slot), ad, 0, first);
          wait_loads_barrier<LOADS>();
          kb = kc;
          kc = kd;
          kd = kn;
        }
      }
      while (kb >= 0) {   // the rest of the walk is the other waves'
        phase_barrier();
        slot = (slot + 1) & 3;
        wait_loads_barrier<LOADS>();
        kb = kc;
        kc = kd;
        kd = kn;
        kn = walk.cursor();
        walk.issue(k_lds((slot + 3) & 3), v_lds((slot + 3) & 3), wave, lane);
      }
      wait_global_loads();   // sets past the end of the walk
      if (wave < NW / 2) phase_barrier();
    }
  }

  float l_sum[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    l_sum[nb] = (l_run[nb][0] + l_run[nb][1]) + (l_run[nb][2] + l_run[nb][3]);
    l_sum[nb] += __shfl_xor(l_sum[nb], 16, 64);
    l_sum[nb] += __shfl_xor(l_sum[nb], 32, 64);
  }
  // SPLIT: the waves' sums meet in LDS (each where its tiles were), and wave w goes on with columns of blocks w DBO ..
  constexpr int DBO = SPLIT ? DB / NW : DB;
  const int col0 = 4 * g + (SPLIT ? 16 * DBO * wave : 0);
  const bool writes_lse = g == 0 && (!SPLIT || wave == 0);
  float lse_before[NB];
  if constexpr (SPLIT) {
    SplitRow* const rows = reinterpret_cast<SplitRow*>(smem + SLOTS * 2 * TILE);
    f32x4* const sums = reinterpret_cast<f32x4*>(smem) + lane;
    constexpr int PER_WAVE = 2 * TILE / 16;
    static_assert(DB * NB * 64 <= PER_WAVE, "a wave's sums fit where its tiles were");
#pragma unroll
    for (int i = 0; i < DB * NB; ++i) sums[wave * PER_WAVE + i * 64] = o[i / NB][i % NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int orow = q_w0 + 16 * nb + r;
      if (g == 0) {
        rows[wave * BQ + 16 * nb + r] = {m_sums[nb], l_sum[nb],
                                         wave == 0 && p.o_acc.ptr && orow < sq ? p.lse_acc.ptr[b * p.lse_acc.sb + hq * p.lse_acc.sh + orow] : 0.f};
      }
    }
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      SplitRow part[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) part[w] = rows[w * BQ + 16 * nb + r];
      lse_before[nb] = part[0].lse_before;
      m_run[nb] = part[0].m;
#pragma unroll
      for (int w = 1; w < NW; ++w) m_run[nb] = fmaxf(m_run[nb], part[w].m);
      l_sum[nb] = 0.f;
#pragma unroll
      for (int i = 0; i < DBO; ++i) o[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {   // (a wave without keys for the row: zeros of weight one or zero)
        const float weight = part[w].m == m_run[nb] ? 1.f : __builtin_amdgcn_exp2f(c * (part[w].m - m_run[nb]));
        l_sum[nb] += weight * part[w].l;
#pragma unroll
        for (int i = 0; i < DBO; ++i) o[i][nb] += weight * sums[w * PER_WAVE + ((wave * DBO + i) * NB + nb) * 64];
      }
    }
  }

  // Epilogue: normalise, Lse in natural-log units, optional online-softmax merge.
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float l_tot = l_sum[nb];
    const int orow = q_w0 + 16 * nb + r;
    if (orow >= sq) continue;
    const bool alive = l_tot != 0.f;   // (zero: no key seen; NaN is seen)
    const float inv = alive ? 1.f / l_tot : 0.f;
    const float lse_cur = alive ? (c * m_run[nb] + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
    if (p.o_part.ptr) {
      const int64_t off = b * p.o_part.sb + (int64_t)orow * p.o_part.ss + hq * p.o_part.sh + col0;
      if (p.o_part.is_f32) {
        float* dst = (float*)p.o_part.ptr + off;
#pragma unroll
        for (int db = 0; db < DBO; ++db) *reinterpret_cast<f32x4*>(dst + 16 * db) = o[db][nb] * inv;
      } else {
        __bf16* dst = (__bf16*)p.o_part.ptr + off;
#pragma unroll
        for (int db = 0; db < DBO; ++db) {
          const f32x4 x = o[db][nb] * inv;
          *reinterpret_cast<bf16x4*>(dst + 16 * db) = bf16x4{(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
        }
      }
      if (writes_lse) p.lse_part.ptr[b * p.lse_part.sb + hq * p.lse_part.sh + orow] = lse_cur;
    }
    if (p.o_acc.ptr && alive) {   // a step that saw no key leaves the running state untouched
      float* lse_ptr = p.lse_acc.ptr + b * p.lse_acc.sb + hq * p.lse_acc.sh + orow;
      const float lse_old = SPLIT ? lse_before[nb] : *lse_ptr;
      const float mm = fmaxf(lse_old, lse_cur);   // finite, or lse_cur is NaN and reaches everything below
      const float e_old = __expf(lse_old - mm), e_cur = __expf(lse_cur - mm);
      const float tot = e_old + e_cur;
      const float lse_new = mm + __logf(tot);
      const float w_old = e_old / tot, w_cur_n = e_cur / tot * inv;
      const bool has_old = lse_old != -INFINITY;
      float* dst = (float*)p.o_acc.ptr + b * p.o_acc.sb + (int64_t)orow * p.o_acc.ss + hq * p.o_acc.sh + col0;
#pragma unroll
      for (int db = 0; db < DBO; ++db) {
        f32x4* q4 = reinterpret_cast<f32x4*>(dst + 16 * db);
        // a running state that is still (anything, -inf) has weight zero and is not read as a number:
        // the buffer may hold whatever it was allocated with (0 * NaN would poison the row)
        f32x4 old = *q4;
        if (!has_old) old = f32x4{0.f, 0.f, 0.f, 0.f};
        *q4 = o[db][nb] * w_cur_n + old * w_old;
      }
      // the four lanes of a row read lse_old above, in lockstep, before this store
      if (writes_lse) *lse_ptr = lse_new;
    }
  }
}

// Query rows of a step that no launched work-group covers (their tiles see no key): the step
// result for them is (0, -inf); the running state is left alone.
__global__ __launch_bounds__(256) void fwd_fill_dead_rows_kernel(FwdParams p, int tile_rows) {
  const int d4 = p.head_dim / 4;
  const int n_tiles = (p.sq + tile_rows - 1) / tile_rows;
  const int64_t total = (int64_t)p.batch * p.sq * p.q_heads * d4;
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int cc = i % d4;
    int64_t rest = i / d4;
    const int hq = rest % p.q_heads;
    rest /= p.q_heads;
    const int row = rest % p.sq;
    const int b = rest / p.sq;
    const int tile = row / tile_rows;
    const bool covered = (tile >= p.q_runs.start[0] && tile < p.q_runs.start[0] + p.q_runs.len[0]) ||
                         (tile >= p.q_runs.start[1] && tile < p.q_runs.start[1] + p.q_runs.len[1]);
    if (covered || tile >= n_tiles) continue;
    const int64_t off = b * p.o_part.sb + (int64_t)row * p.o_part.ss + hq * p.o_part.sh + cc * 4;
    if (p.o_part.is_f32) {
      *reinterpret_cast<f32x4*>((float*)p.o_part.ptr + off) = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
      *reinterpret_cast<bf16x4*>((__bf16*)p.o_part.ptr + off) = bf16x4{(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
    }
    if (cc == 0) p.lse_part.ptr[b * p.lse_part.sb + hq * p.lse_part.sh + row] = -INFINITY;
  }
}

// Whether the waves of a work-group share 32 query rows and deal the key tiles among themselves (SPLIT).  A launch of few query
// tiles is as long as its longest walk, and shared out to four waves that walk is four times shorter, on eight (d = 64: four)
// times as many work-groups.  A wave alone with its tiles, two products and the softmax one after the other, takes 1.3 (d = 64: 2.3) times as long
// for one as the kernel whose waves take turns, and brings every tile for 32 rows, so that the other one is faster where there are more than
// about two work-groups a CU whose walks are all as long as the longest; where they are uneven, work-groups times their mean walk over the longest
// one count, up to four a CU under a causal mask.  us of a step by the kernels of one walk a wave and by this one, d = 128 (d = 64), with that count: full
// 2 x 256 rows (16) 17.7, 8.3 (8.6, 6.7); 4 x 1024 (128) 33, 15 (18.5, 10.8); 1 x 8192 (256) 179, 70 (109, 47); 16 x 1024 (512) 34.5, 27.8 (19.3,
// 13.8); 20 x 1024 (640) 36, 40 (19.5, 20.7); 32 x 1000 (1024) 38, 54 (20, 25); causal 1 x 16384 (256) 340, 138 (210, 96); 1 x 32768 (512) 667, 497 (414,
// 239); 16 x 2048 (528) 56.5, 58.7 (33, 28); 48 x 512, two steps (576) 41, 50 (22, 28); 1 x 49546 (775) 1000, 1108 (643, 512); window of 1000 tokens 4 x 4096 (480) 43,
// 34 (24, 17); 8 x 4096 (960) 47, 63 (25, 29); zigzag with a window, 32 heads, the shard one place ahead: 16384 rows, window 6000 (3040) 347, 692 (217, 316); 65536
// rows, window 30000 (15040) 6840, 13600 (4220, 8630).
// At d = 64 two work-groups share a CU, and of a second, part-empty round each has the CU to itself and is faster: with walks that
// are long beside what a work-group starts and ends with, the line lies higher.  d = 64: 64 tiles a walk, 5 x 4096 rows (640) 59, 55; 6 x 4096 (768) 60, 56; 8 x
// 4096 (1024) 60, 65; causal 12 x 4096 (780) 64, 59; 16 x 4096 (1040) 64, 78; 1 x 60000 (940) 786, 718; 16 tiles, 17 x 1024 (544) 19.8, 21.5.  d = 128: causal
// 8 x 4096 (520) 97, 88; 1 x 17000 (532) 359, 375; 5 x 4096 (640) 98, 105.
template <int D>
static int64_t split_load(int64_t longest) {
  return D == 128 ? 520 : longest < 64 ? 544 : 800;
}
template <int D>
static bool split_walks(const FwdParams& p) {
  const Walks w = q_walks(p.step, p.n_steps, p.sq, kSplitBQ);
  return w.longest > 0 && (int64_t)p.batch * p.q_heads * w.total <= split_load<D>(w.longest) * w.longest;
}
template <int D, bool SPLIT>
static hipError_t launch_fwd_t(FwdParams& p, hipStream_t stream, LaunchLog* log) {
  constexpr int BQ = SPLIT ? kSplitBQ : kFwdBQ<D>, NW = SPLIT ? kSplitWaves : kFwdWaves<D>;
  constexpr int LDS = (SPLIT ? NW * (2 * 64 * 2 * D + BQ * (int)sizeof(SplitRow)) + SplitPosts::BYTES : kFwdSlots<D> * 2 * 64 * 2 * D) + kMaxBlockCacheTiles;
  p.q_runs = nonempty_q_runs(p.step, p.n_steps, p.sq, BQ);
  if (log) {
    if (p.q_runs.total() > 0) log->push_back(SPLIT ? BURST_KERNEL_DEALT : 0);
    return hipSuccess;
  }
  const int n_tiles = (p.sq + BQ - 1) / BQ;
  if (p.o_part.ptr && p.q_runs.total() < n_tiles) {
    const int64_t total = (int64_t)p.batch * p.sq * p.q_heads * (p.head_dim / 4);
    const int64_t blocks = (total + 255) / 256;
    hipLaunchKernelGGL(fwd_fill_dead_rows_kernel, dim3((int)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, stream, p, BQ);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (p.q_runs.total() == 0) return hipSuccess;
  const int n_keys = p.batch * p.kv_heads, group = p.q_heads / p.kv_heads;
  p.q_side_by_side = q_side_by_side(p.step, p.n_steps, p.sq, n_keys, group, p.q_runs, BQ);
  const int grid = mapped_grid(n_keys, group, p.q_runs.total());
  constexpr int NT = 64 * NW;
  if (p.step[0].mask.blk) hipLaunchKernelGGL((step_fwd_kernel<D, NW, true, false, SPLIT>), dim3(grid), dim3(NT), LDS, stream, p);
  else if (p.n_steps > 1) hipLaunchKernelGGL((step_fwd_kernel<D, NW, false, true, SPLIT>), dim3(grid), dim3(NT), LDS, stream, p);
  else hipLaunchKernelGGL((step_fwd_kernel<D, NW, false, false, SPLIT>), dim3(grid), dim3(NT), LDS, stream, p);
  return hipGetLastError();
}
template <int D>
static hipError_t launch_fwd_steps(FwdParams& p, hipStream_t stream, LaunchLog* log) {
  return split_walks<D>(p) ? launch_fwd_t<D, true>(p, stream, log) : launch_fwd_t<D, false>(p, stream, log);
}

// With the fused merge and no separate step result, a key axis longer than two ranges is cut into ranges, each walked as
// a step of its own: the same online-softmax merge the ring applies from step to step, so the result is the step's up to
// rounding.  The step result itself (o_part, lse_part) cannot be cut this way and is always one launch.
template <int D>
static hipError_t launch_fwd_groups(const FwdParams& p0, const FwdStep* steps, int n, hipStream_t stream, LaunchLog* log) {
  FwdParams p = p0;
  if (!p.o_acc.ptr || p.o_part.ptr) {
    p.n_steps = 1;
    p.step[0] = steps[0];
    return launch_fwd_steps<D>(p, stream, log);
  }
  std::vector<FwdStep> parts;
  for (int i = 0; i < n; ++i) {
    const MaskDev& mk = steps[i].mask;
    const std::vector<RowRange> ranges = chunk_ranges(mk.k_nseg, mk.k_seg_len, steps[i].sk, mk.blk ? mk.blk_k : 0);
    for (const RowRange& rg : ranges) {
      FwdStep st = steps[i];
      if (ranges.size() > 1) {
        st.mask = sub_mask<false>(mk, rg.r0, rg.r1);
        st.sk = rg.r1 - rg.r0;
        offset_rows(st.k, rg.r0);
        offset_rows(st.v, rg.r0);
      }
      parts.push_back(st);
    }
  }
  return for_step_groups(parts, p.sq, p.batch * p.q_heads, [&](int first, int end) {
    p.n_steps = end - first;
    std::copy(parts.begin() + first, parts.begin() + end, p.step);
    return launch_fwd_steps<D>(p, stream, log);
  });
}

hipError_t launch_steps_fwd(const FwdParams& p, const FwdStep* steps, int n, hipStream_t stream, LaunchLog* log) {
  if (p.head_dim == 128) return launch_fwd_groups<128>(p, steps, n, stream, log);
  return launch_fwd_groups<64>(p, steps, n, stream, log);
}

}  // namespace burst
