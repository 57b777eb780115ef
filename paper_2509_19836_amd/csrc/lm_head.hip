// Sequence-level fusion of the LM head and the loss function (Sec. 3.3, Eq. 9, Alg. 3).
//
// Per sequence tile of B_s tokens, four launches:
//   1. lm_logits_kernel       Logits^T tile = W_head H_i^T on the matrix cores (bf16 in, fp32 out).
//                             Computed transposed so that a lane owns a token: the per-token
//                             (max, sum of exp) over 128 words starts as a reduction over
//                             a lane's own registers, as in the attention forward.  The fp32 logits of
//                             the tile go to the workspace (the algorithm keeps them between its two
//                             sweeps over the vocabulary); the partial (max, sum) pairs go to a side array.
//   2. lm_loss_dlogits_kernel one work-group per token: merges the partial pairs into Lse_i, writes
//                             the loss, then streams the token's logits once and writes
//                             grad_scale * (exp(Logits - Lse) - E) as bf16 (HBM-bound).
//   3. lm_dh_kernel           dH_i  = dLogits W_head          (contraction over the vocabulary)
//   4. lm_transpose_h_kernel + lm_dw_kernel
//                             dW^T += H_i^T dLogits           (contraction over the tile's tokens)
// The three GEMMs share one main loop (LmGemm below), or where tiles of 256 x 256 are few or short LmGemmSmall (lm_plan).  An operand whose contraction index is the storage row is
// read with the transposing LDS read; only H_i, a few MB per sequence tile, is ever transposed in memory.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "mfma16.hpp"

namespace burst {

namespace {

// Output tile of a work-group of eight waves, and the k-tile; 128 accumulator registers per wave.
constexpr int kLmBM = 256, kLmBN = 256, kLmBK = 64, kLmThreads = 512;

// One GEMM operand: where its k-tiles come from and how they lie in LDS (X rows or columns of 128 bytes: 32 KiB for the 256 of an
// output tile of eight waves, 16 KiB for the 128 of one of four).  A k-tile is four direct loads per wave.
//   COLS = false: storage [x][k], k contiguous.  LDS: [X x][64 k].  lim = valid storage rows; rows beyond are
//                 read as the last one (folded into the per-lane offsets once).
//   COLS = true : storage [k][x], x contiguous.  LDS: X / 128 tiles [64 k][128 x], the k rows permuted so that the
//                 transposing read, which hands out rows 16 (e / 4) + 4 g + e % 4 of 32, gives k = 8 g + e as the
//                 row-wise operand has it.  lim = valid k rows; a k-tile that reaches past them reads copies of
//                 the last one.
template <bool COLS, int X, int NW>   // X rows or columns of the output tile, brought by NW waves
struct LmOperand {
  static constexpr int N = 4, BYTES = X * kLmBK * 2;
  static_assert(BYTES == N * NW * 1024, "four loads per wave");
  using Rows = DirectStager<64, X, NW>;
  using Cols = DirectStager<128, kLmBK, NW>;   // one of the X / 128 tiles
  Rows rows;
  uint32_t col_off[Cols::N];
  const char* tile;     // k-tile to ask for
  int64_t ld, step;
  int left, valid;      // k-tiles behind it; valid k rows from its first one on (COLS)

  __device__ __forceinline__ void init(const __bf16* ptr, int64_t ld_, int lim, int x0, int nk, int wave, int lane) {
    ld = ld_;
    left = nk - 1;
    tile = reinterpret_cast<const char*>(COLS ? ptr + x0 : ptr + (int64_t)x0 * ld);
    step = COLS ? kLmBK * ld * 2 : kLmBK * 2;
    if (COLS) {
      valid = lim;
      offsets(wave, lane);
    } else {
      rows.clamp(ld, min(X, lim - x0), wave, lane);
    }
  }
  __device__ __forceinline__ void offsets(int wave, int lane) {
#pragma unroll
    for (int i = 0; i < Cols::N; ++i) {
      const int at = (i * NW + wave) * Cols::RPI + lane / 16;   // row in LDS
      const int k = (at & 32) + 8 * ((at >> 2) & 3) + 4 * ((at >> 4) & 1) + (at & 3);
      col_off[i] = 2u * ((uint32_t)min(k, valid - 1) * (uint32_t)ld + (uint32_t)(((lane % 16) ^ swz<128>(at)) * 8));
    }
  }
  // To the next k-tile; on the last one the cursor stays (that tile is then asked for again and not read)
  __device__ __forceinline__ void next(int wave, int lane) {
    const int move = min(left, 1);   // (arithmetic on 0 / 1: the compiler keeps selected addresses in vector registers)
    left -= move;
    tile += step & -(int64_t)move;
    if (COLS) {
      valid -= kLmBK * move;
      if (valid < kLmBK) offsets(wave, lane);
    }
  }
  __device__ __forceinline__ void load(int i, uint32_t lds, int wave) const {
    constexpr int PER = Cols::N;   // loads of a tile
    if (COLS) load_to_lds(tile + (i / PER) * 256, col_off[i % PER], lds + (i / PER) * Cols::BYTES + ((i % PER) * NW + wave) * 1024);
    else rows.load_one(tile, i, lds, wave);
  }
};

// The main loop.  The matrix pipe bounds it (2048 clocks per k-tile and SIMD, against 1536 clocks of LDS reads and
// 512 of LDS writes per CU); what is to be avoided is waiting at the barriers.
//  - 16x16x32 MFMAs, k-tiles by direct global -> LDS loads: no staging registers, no LDS store instructions.
//  - A k-tile is two phases, each over one half of the 256 A rows and all of B (a wave: 64 of the 128 A rows against
//    its 64 B columns, 32 MFMAs).  B stays in registers for the second phase, so B and the lower half of A are free
//    after the first one: their successors of k-tile t + 2 are asked for in phase 2 of t, those of the upper half of
//    A in phase 1 of t + 1, and every load has two phases until its tile is announced by a barrier, a full phase
//    before it is read.  The first operands of a phase are therefore fetched in the one before, across the barrier.
// 8192 tokens, d = 4096, 32000 words, fastest launch of a run: logits 1.72 ms (1250 TFLOP/s), dH 1.51 (1420), dW 1.69
// (1270); with 32x32x16 MFMAs, tiles staged through registers and one barrier per k-tile: 2.10, 1.86, 2.09.  (Means of a run, in which
// the clock falls: 1.78, 1.67, 1.83.  Single launches with counters: 1.81 ms at 68 % busy and 1.66 GHz, 1.81 at 78 % and
// 1.45, 1.93 at 69 % and 1.54.)  A k-tile takes 1.51 us;
// the rest of logits and dW (13 and 23 us per output tile) is their fp32 output, which all CUs write at the same time.
template <bool B_COLS>
struct LmGemm {
  using OpA = LmOperand<false, kLmBM, 8>;
  using OpB = LmOperand<B_COLS, kLmBN, 8>;
  static constexpr int BM = kLmBM, BN = kLmBN, HALVES = 2, THREADS = kLmThreads;
  static constexpr int SLOT = OpA::BYTES + OpB::BYTES, LDS = 2 * SLOT, AHEAD = 3;
  f32x4 acc[2][4][4];   // [half][mb][nb]: rows 128 half + 64 wm + 16 mb + 4 g + v, column 64 wn + 16 nb + r
  bf16x8 bf[2][4];      // [k-step][nb]
  bf16x8 first[AHEAD];
  OperandAddr<64> ad;
  OperandAddr<128> adc;

  __device__ __forceinline__ bf16x8 a_operand(uint32_t slot, int half, int wm, int i) const {   // i: 4 k-steps + mb
    return rows_operand<64>(slot + half * (OpA::BYTES / 2) + wm * (64 * 128), ad, 16 * (i % 4), i / 4);
  }
  __device__ __forceinline__ bf16x8 b_operand(uint32_t slot, int wn, int ks, int nb) const {
    if (B_COLS) return cols_operand<128>(slot + OpA::BYTES + (wn >> 1) * OpB::Cols::BYTES, adc, 32 * ks, nb);
    return rows_operand<64>(slot + OpA::BYTES + wn * (64 * 128), ad, 16 * nb, ks);
  }
  // The 32 MFMAs of a phase, hook(i) behind the four of operand i.  The next phase reads half HALF ^ 1 from slot `next`.
  template <int HALF, class Hook>
  __device__ __forceinline__ void phase(uint32_t slot, uint32_t next, int wm, int wn, Hook&& hook) {
    bf16x8 a[8 + AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) a[i] = first[i];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      a[i + AHEAD] = i + AHEAD < 8 ? a_operand(slot, HALF, wm, i + AHEAD) : a_operand(next, HALF ^ 1, wm, i + AHEAD - 8);
      if (HALF == 0 && (i == 1 || i == 2)) {   // second k-step of this tile
#pragma unroll
        for (int j = 0; j < 2; ++j) bf[1][2 * (i - 1) + j] = b_operand(slot, wn, 1, 2 * (i - 1) + j);
      }
      if (HALF == 1 && (i == 4 || i == 5)) {   // first k-step of the next tile
#pragma unroll
        for (int j = 0; j < 2; ++j) bf[0][2 * (i - 4) + j] = b_operand(next, wn, 0, 2 * (i - 4) + j);
      }
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) acc[HALF][i % 4][nb] = mfma16(a[i], bf[i / 4][nb], acc[HALF][i % 4][nb]);
      hook(i);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) first[i] = a[8 + i];
  }

  // nk >= 1 k-tiles, of which a and b point at the first
  __device__ __forceinline__ void run(char* smem, OpA& a, OpB& b, int nk, int wm, int wn, int wave, int lane) {
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_bytes)smem;
    ad.init(lane);
    adc.init(lane);
    adc.cols ^= (uint32_t)(wn & 1) << 7;   // column blocks 4 .. 7 of the tile
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[half][mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto load_b_lower_a = [&](int i, uint32_t slot) {
      if (i < 4) b.load(i, slot + OpA::BYTES, wave);
      else a.load(i - 4, slot, wave);
    };
    wait_global_loads();
#pragma unroll
    for (int i = 0; i < 6; ++i) load_b_lower_a(i, lds0);
#pragma unroll
    for (int i = 2; i < 4; ++i) a.load(i, lds0, wave);
    a.next(wave, lane);
    b.next(wave, lane);
#pragma unroll
    for (int i = 0; i < 6; ++i) load_b_lower_a(i, lds0 + SLOT);
    wait_loads_barrier<6>();               // tile 0
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) bf[0][nb] = b_operand(lds0, wn, 0, nb);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) first[i] = a_operand(lds0, 0, wm, i);
    __builtin_amdgcn_s_waitcnt(0xc07f);    // lgkmcnt(0): lets the compiler count the LDS reads at the head of the loop
    uint32_t slot = lds0, other = lds0 + SLOT;
    for (int t = 0; t < nk; ++t) {
      phase<0>(slot, slot, wm, wn, [&](int i) {
        if (i >= 2 && i < 4) a.load(i, other, wave);         // upper half of A, tile t + 1
      });
      a.next(wave, lane);
      b.next(wave, lane);
      wait_loads_barrier<2>();             // B and lower half of A, tile t + 1
      phase<1>(slot, other, wm, wn, [&](int i) {
        if (i < 6) load_b_lower_a(i, slot);                  // tile t + 2
      });
      wait_loads_barrier<6>();             // upper half of A, tile t + 1
      const uint32_t x = slot;
      slot = other;
      other = x;
    }
    wait_global_loads();                   // tiles past the end
  }
};

// Output tiles of 128 x 128 by four waves, two work-groups per CU, for short contractions and for few output tiles: a work-group's first
// loads and its fp32 output, which a CU with one work-group waits for at each end, pass while the other one multiplies.  Where the
// contraction is long this is the slower loop: it brings twice the bytes, and reads a third more from LDS, per product.
// Tile t + 2 is asked for when all waves have left tile t; the other work-group's matrix phases cover its way.
template <bool B_COLS>
struct LmGemmSmall {
  static constexpr int BM = 128, BN = 128, HALVES = 1, THREADS = 256;
  using OpA = LmOperand<false, BM, 4>;
  using OpB = LmOperand<B_COLS, BN, 4>;
  static constexpr int SLOT = OpA::BYTES + OpB::BYTES, LDS = 2 * SLOT;
  f32x4 acc[1][4][4];   // [0][mb][nb]: rows 64 wm + 16 mb + 4 g + v, column 64 wn + 16 nb + r

  __device__ __forceinline__ void run(char* smem, OpA& a, OpB& b, int nk, int wm, int wn, int wave, int lane) {
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_bytes)smem;
    OperandAddr<64> ad;
    OperandAddr<128> adc;
    ad.init(lane);
    adc.init(lane);
    adc.cols ^= (uint32_t)wn << 7;         // column blocks 4 .. 7 of the tile
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[0][i / 4][i % 4] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto ask = [&](uint32_t slot) {
#pragma unroll
      for (int i = 0; i < 4; ++i) a.load(i, slot, wave);
#pragma unroll
      for (int i = 0; i < 4; ++i) b.load(i, slot + OpA::BYTES, wave);
      a.next(wave, lane);
      b.next(wave, lane);
    };
    wait_global_loads();
    ask(lds0);
    ask(lds0 + SLOT);
    uint32_t slot = lds0, other = lds0 + SLOT;
    for (int t = 0; t < nk; ++t) {
      wait_loads_barrier<8>();             // tile t
      bf16x8 x[2][4], y[2][4];             // [k-step]: A, B
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[ks][i] = rows_operand<64>(slot + wm * (64 * 128), ad, 16 * i, ks);
          y[ks][i] = B_COLS ? cols_operand<128>(slot + OpA::BYTES, adc, 32 * ks, i) : rows_operand<64>(slot + OpA::BYTES + wn * (64 * 128), ad, 16 * i, ks);
        }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[0][i / 4][i % 4] = mfma16(x[ks][i / 4], y[ks][i % 4], acc[0][i / 4][i % 4]);
      phase_barrier();                     // all waves have left the slot
      ask(slot);
      const uint32_t z = slot;
      slot = other;
      other = z;
    }
    wait_global_loads();                   // tiles past the end
  }
};
template <bool SMALL, bool B_COLS>
using LmGemmOf = std::conditional_t<SMALL, LmGemmSmall<B_COLS>, LmGemm<B_COLS>>;

// Work-group -> output tile and, where the contraction is split, its part of the k-tiles.  Work-group n runs on XCD
// n mod 8.
//  - More than one work-group per CU (kLmOneRound): each XCD takes groups of 4 x 8 tiles (one per CU), so the 32
//    work-groups that share an L2 at a time read 4 + 8 operand panels.
//  - Else every XCD takes an eighth of the tiles, neighbours in m first: what counts is that no CU gets two while
//    another has none (16 tiles of dH for 256 tokens are one group of eight on two XCDs).
constexpr int kLmOneRound = 256;   // (128 x 128 tiles: twice as many)
template <class G>
__device__ __forceinline__ bool lm_tile(int bid, int TM, int TN, int splits, int& tm, int& tn, int& split) {
  const int xcd = bid & 7, slot = bid >> 3, total = TM * TN * splits;
  split = 0;
  if (total <= kLmOneRound * (G::HALVES == 1 ? 2 : 1)) {
    const int per = (total + 7) / 8, i = xcd * per + slot;
    if (slot >= per || i >= total) return false;
    split = i / (TM * TN);
    const int t = i - split * (TM * TN);
    tn = t / TM;
    tm = t - tn * TM;
    return true;
  }
  const int groups_m = (TM + 3) / 4, groups_n = (TN + 7) / 8;
  const int group = (slot >> 5) * 8 + xcd, within = slot & 31;
  if (group >= groups_m * groups_n) return false;
  const int gm = group % groups_m, gn = group / groups_m;
  tm = gm * 4 + (within & 3);
  tn = gn * 8 + (within >> 2);
  return tm < TM && tn < TN;
}
int lm_grid(int TM, int TN, int splits, bool small) {
  const int total = TM * TN * splits;
  if (total <= kLmOneRound * (small ? 2 : 1)) return (total + 7) / 8 * 8;
  const int groups = ((TM + 3) / 4) * ((TN + 7) / 8);
  return (groups + 7) / 8 * 8 * 32;
}

// dH contracts over the vocabulary, hundreds of k-tiles, and has few output tiles when the sequence tile is short: its
// k-tiles are then dealt to `splits` work-groups per output tile, as many as fill the CUs, which leave fp32 partial
// sums for lm_dh_sum_kernel in the logits buffer (read for the last time before).  Bounds: that buffer, and 16 k-tiles
// a part, below which starting a work-group and the extra pass over the partial sums cost more than they give.
// 256 tokens, d = 4096, 32000 words (16 output tiles, 7 parts): dH 650 -> 117 us with the sum; the call over 1000
// tokens in such tiles 3866 -> 1887 us.
int lm_dh_splits(const LmHeadParams& p, int TM, int TN, bool small) {
  const int64_t fits = (int64_t)p.tile_tokens * p.v_pad / ((int64_t)TM * (small ? 128 : kLmBM) * p.d_model);
  const int64_t s = std::min<int64_t>({kLmOneRound * (small ? 2 : 1) / (TM * TN), fits, p.vocab / (16 * kLmBK)});
  return (int)std::max<int64_t>(s, 1);
}

// The logits contract over the hidden dimension and have few output tiles when the sequence tile or the vocabulary is short:
// the k-tiles are then dealt to as many work-groups per output tile as fill the CUs, which leave partial logits, one
// array of the tile's rows (up to a multiple of 256) behind the other in the logits buffer, for lm_loss_dlogits_kernel to add
// up.  Bounds: that buffer, 16 k-tiles a part, and kLmSplitWords words times parts, beyond which the parts ask for W faster
// than memory gives it (a part's k-tile takes 1.5 us, its 32 KiB of W at 5 TB/s over all of them as long).  The whole call, us,
// without and with: d = 4096, 100 tokens: 8000 words (4 parts) 150, 108, 32000 (2, against the bound) 353, 366; 300 x 16000 (2)
// 261, 241; 700 x 8000, d = 5120 (2) 259, 230; 64 x 20000, d = 2048 (2) 131, 119; 70 x 30000 (2) 368, 342; without a workspace
// 200 x 20000 (3) 315, 248, 500 x 10000 (3) 255, 189.
constexpr int kLmSplitWords = 60000;
int lm_logit_splits(const LmHeadParams& p, int TM, int TN) {
  const int64_t s = std::min<int64_t>({kLmOneRound / (TM * TN), p.tile_tokens / (TN * kLmBN), p.d_model / (16 * kLmBK), kLmSplitWords / p.vocab});
  return (int)std::max<int64_t>(s, 1);
}

// Tiles of one of the three products over a sequence tile
struct LmPlan {
  int TM, TN, splits;
  bool small;   // tiles of 128 x 128 (LmGemmSmall)
  int tile() const { return small ? 128 : kLmBM; }
  // Tenths of a microsecond, by rounds of work-groups: 1.5 us a k-tile and 14 us for first loads and output of a 256 x 256 tile; 1.1 and
  // 5 us of two work-groups with a 128 x 128 tile each.
  int64_t time(int nk) const {
    const int64_t groups = (int64_t)TM * TN * splits, parts = (nk + splits - 1) / splits;
    return small ? (groups + 2 * kLmOneRound - 1) / (2 * kLmOneRound) * (11 * parts + 50) : (groups + kLmOneRound - 1) / kLmOneRound * (15 * parts + 140);
  }
};
// The small tiles where they are clearly ahead by that: a tenth for the logits, a fifth for the other two, whose small tiles a long run of rounds
// holds up more than it says (dW of 281 tokens x 73783 words, d = 768, 0.85 of the time by it: 9 us slower).  The whole call, us, with
// 256 x 256 tiles and with small ones for that product alone: logits, d = 768, 2426 tokens x 8354 words (2 rounds, 3) 193, 169; 281 x 73783 297,
// 278; d = 1024, 242 x 8216 87, 73; d = 2048, 64 x 113750 603, 555; against the rule: d = 768, 2048 x 60455 787, 863; d = 4096, 1000 x 32000 767, 854.
// dW: d = 768, 2426 x 8354 (99 tiles) 193, 178; 2048 x 9304 164, 152; d = 2048, 129 x 17229 123, 118; against: d = 512, 4096 x 29660 581, 627.  dH:
// d = 2560, 207 x 10874 (4 parts, by the room for them) 166, 146; d = 1024, 242 x 8216 87, 78; against: d = 768, 635 x 52993 311, 316.
LmPlan lm_plan(const LmPlan& big, const LmPlan& small, int nk, int tenths) { return 10 * small.time(nk) <= tenths * big.time(nk) ? small : big; }
LmPlan lm_plan_logits(const LmHeadParams& p, int n_rows) {
  LmPlan big{p.v_pad / kLmBM, (n_rows + kLmBN - 1) / kLmBN, 1, false};
  big.splits = lm_logit_splits(p, big.TM, big.TN);
  return lm_plan(big, LmPlan{(p.vocab + 127) / 128, (n_rows + 127) / 128, 1, true}, p.d_model / kLmBK, 9);
}
LmPlan lm_plan_dh(const LmHeadParams& p, int n_rows) {
  LmPlan big{(n_rows + kLmBM - 1) / kLmBM, p.d_model / kLmBN, 1, false}, small{(n_rows + 127) / 128, p.d_model / 128, 1, true};
  big.splits = lm_dh_splits(p, big.TM, big.TN, false);
  small.splits = lm_dh_splits(p, small.TM, small.TN, true);
  return lm_plan(big, small, (p.vocab + kLmBK - 1) / kLmBK, 8);
}
LmPlan lm_plan_dw(const LmHeadParams& p, int n_rows) {
  return lm_plan(LmPlan{p.d_model / kLmBM, p.v_pad / kLmBN, 1, false}, LmPlan{p.d_model / 128, (p.vocab + 127) / 128, 1, true}, (n_rows + kLmBK - 1) / kLmBK, 8);
}

// (max, sum of exp(x - max)) pairs combine like the log-sum-exp merge of the attention forward.
__device__ __forceinline__ void lm_combine(float& m, float& l, float m2, float l2) {
  const float mm = fmaxf(m, m2);
  l = (mm == -INFINITY) ? 0.f : l * __expf(m - mm) + l2 * __expf(m2 - mm);
  m = mm;
}

// ---------------------------------------------------------------------------------------------
// 1. Logits^T tile (rows: words, columns: tokens of the sequence tile), Alg. 3 forward sweep.
// ---------------------------------------------------------------------------------------------
template <bool SMALL>
__global__ __launch_bounds__((LmGemmOf<SMALL, false>::THREADS), 2) void lm_logits_kernel(LmHeadParams p, int s0, int n_rows, int TM, int TN, int splits) {
  using G = LmGemmOf<SMALL, false>;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int tm, tn, split;
  if (!lm_tile<G>(blockIdx.x, TM, TN, splits, tm, tn, split)) return;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;
  const int m0 = tm * G::BM, n0 = tn * G::BN, nk_all = p.d_model / kLmBK;
  const int kt0 = nk_all * split / splits, nk = nk_all * (split + 1) / splits - kt0, k0 = kt0 * kLmBK;
  typename G::OpA a;
  typename G::OpB b;
  a.init(p.w + k0, p.ld_w, p.vocab, m0, nk, wave, lane);
  b.init(p.h + (int64_t)s0 * p.ld_h + k0, p.ld_h, n_rows, n0, nk, wave, lane);
  G gemm;
  gemm.run(smem, a, b, nk, wm, wn, wave, lane);

  const int word0 = m0 + wm * 64 + 4 * g;              // first word of the lane
  if (splits > 1) {
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      float* dst = p.logits + ((int64_t)split * TN * G::BN + n0 + wn * 64 + 16 * nb + r) * p.v_pad + word0;
#pragma unroll
      for (int i = 0; i < 4 * G::HALVES; ++i) *reinterpret_cast<f32x4*>(dst + 128 * (i / 4) + 16 * (i % 4)) = gemm.acc[i / 4][i % 4][nb];
    }
    return;
  }
  // (max, sum of exp) of a token over 128 consecutive words, from the 16 words of each of eight lanes in two waves: the same sums in the
  // same order for either tile, so that Lse does not depend on which of them a sequence tile takes.
  constexpr int PITCH = 9;                 // pairs of a token and 128 words: eight, and one to spread the banks
  float2* const pairs = reinterpret_cast<float2*>(smem);
  float2 lane_pair[G::HALVES][4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) {
    const int token = n0 + wn * 64 + 16 * nb + r;      // < tile_tokens: the tile count covers n_rows only
    float* dst = p.logits + (int64_t)token * p.v_pad + word0;
#pragma unroll
    for (int half = 0; half < G::HALVES; ++half) {
      float mx = -INFINITY;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        f32x4& x = gemm.acc[half][mb][nb];
        *reinterpret_cast<f32x4*>(dst + 128 * half + 16 * mb) = x;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          x[v] = word0 + 128 * half + 16 * mb + v < p.vocab ? x[v] : -INFINITY;   // padding words stay out of Lse
          mx = fmaxf(mx, x[v]);
        }
      }
      const float from = mx == -INFINITY ? 0.f : mx;   // (words all at -inf: no share, and a NaN among them, which the maximum leaves out, stays one)
      float sum = 0.f;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int v = 0; v < 4; ++v) sum += __expf(gemm.acc[half][mb][nb][v] - from);
      lane_pair[half][nb] = float2{mx, sum};
    }
  }
  phase_barrier();                         // all waves have left the tiles (the logits' stores go on)
#pragma unroll
  for (int i = 0; i < 4 * G::HALVES; ++i) pairs[((i / 4) * G::BN + wn * 64 + 16 * (i % 4) + r) * PITCH + 4 * wm + g] = lane_pair[i / 4][i % 4];
  stores_barrier<0>();
  if (tid >= G::HALVES * G::BN) return;
  float2 x[8];
  float mx = -INFINITY, sum = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[i] = pairs[tid * PITCH + i];
    mx = fmaxf(mx, x[i].x);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) sum += x[i].x == mx ? x[i].y : x[i].y * __expf(x[i].x - mx);
  p.part[(int64_t)(tm * G::HALVES + tid / G::BN) * p.tile_tokens + n0 + tid % G::BN] = float2{mx, sum};
}

// ---------------------------------------------------------------------------------------------
// 2. Lse_i, loss_i and dLogits of one token per work-group (Alg. 3: the loss line and the first
//    two lines of the backward sweep).  Rows n_rows .. gridDim.x-1 are zero-filled: they pad the
//    contraction of the dW GEMM.
// ---------------------------------------------------------------------------------------------
// SPLIT: the logits come as `splits` partial sums, `part` rows apart; their sum goes where the first of them was.
constexpr int lm_loss_threads(bool split) { return split ? 1024 : 256; }   // (few tokens: more of a row's loads in flight)
template <bool SPLIT>
__global__ __launch_bounds__(lm_loss_threads(SPLIT)) void lm_loss_dlogits_kernel(LmHeadParams p, int s0, int n_rows, int want_grad, int n_part, int splits, int part) {
  constexpr int NT = lm_loss_threads(SPLIT), STEP = 8 * NT;
  __shared__ float red_m[NT / 64], red_l[NT / 64], target;
  const int i = blockIdx.x, tid = threadIdx.x;
  __bf16* drow = p.dlogits + (int64_t)i * p.v_pad;
  const bf16x8 zero8 = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
  if (i >= n_rows) {
    for (int j = tid * 8; j < p.v_pad; j += STEP) *reinterpret_cast<bf16x8*>(drow + j) = zero8;
    return;
  }
  float m = -INFINITY, l = 0.f;
  float* lrow = p.logits + (int64_t)i * p.v_pad;
  const int64_t y = p.y[s0 + i];
  const bool ok = y >= 0 && y < p.vocab;
  if (SPLIT) {
    for (int j = tid * 8; j < p.v_pad; j += STEP) {
      f32x4 x[2] = {*reinterpret_cast<const f32x4*>(lrow + j), *reinterpret_cast<const f32x4*>(lrow + j + 4)};
      for (int s = 1; s < splits; ++s) {
        const float* other = lrow + (int64_t)s * part * p.v_pad + j;
        x[0] += *reinterpret_cast<const f32x4*>(other);
        x[1] += *reinterpret_cast<const f32x4*>(other + 4);
      }
      *reinterpret_cast<f32x4*>(lrow + j) = x[0];
      *reinterpret_cast<f32x4*>(lrow + j + 4) = x[1];
      float mx = -INFINITY, sum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (j + e == y) target = x[e / 4][e % 4];
        if (j + e < p.vocab) mx = fmaxf(mx, x[e / 4][e % 4]);   // padding words stay out of Lse
      }
      // eight words at -inf (masked, or past the fp32 range) have no share: from zero their exponentials are zero, and a NaN
      // among them, which the maximum leaves out, stays one
      const float from = mx == -INFINITY ? 0.f : mx;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (j + e < p.vocab) sum += __expf(x[e / 4][e % 4] - from);
      if (j < p.vocab) lm_combine(m, l, mx, sum);
    }
  } else {
    for (int pp = tid; pp < n_part; pp += NT) {
      const float2 x = p.part[(int64_t)pp * p.tile_tokens + i];
      lm_combine(m, l, x.x, x.y);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) lm_combine(m, l, __shfl_xor(m, off), __shfl_xor(l, off));
  if ((tid & 63) == 0) {
    red_m[tid >> 6] = m;
    red_l[tid >> 6] = l;
  }
  __syncthreads();
  m = red_m[0];
  l = red_l[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) lm_combine(m, l, red_m[w], red_l[w]);
  const float lse = m + __logf(l);
  if (tid == 0) {
    p.loss[s0 + i] = ok ? lse - (SPLIT ? target : lrow[ok ? y : 0]) : 0.f;
    if (p.lse) p.lse[s0 + i] = lse;
  }
  if (!want_grad) return;
  if (!ok) {
    for (int j = tid * 8; j < p.v_pad; j += STEP) *reinterpret_cast<bf16x8*>(drow + j) = zero8;
    return;
  }
  const int yi = (int)y;
  const float gs = p.grad_scale;
  for (int j = tid * 8; j < p.v_pad; j += STEP) {
    const f32x4 x0 = *reinterpret_cast<const f32x4*>(lrow + j), x1 = *reinterpret_cast<const f32x4*>(lrow + j + 4);
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = e < 4 ? x0[e] : x1[e - 4];
      const float g = gs * (__expf(x - lse) - (j + e == yi ? 1.f : 0.f));
      out[e] = (__bf16)(j + e < p.vocab ? g : 0.f);
    }
    *reinterpret_cast<bf16x8*>(drow + j) = out;
  }
}

// ---------------------------------------------------------------------------------------------
// 3. dH_i = dLogits W_head (rows: tokens, columns: hidden, contraction: words).
// ---------------------------------------------------------------------------------------------
template <bool SMALL>
__global__ __launch_bounds__((LmGemmOf<SMALL, true>::THREADS), 2) void lm_dh_kernel(LmHeadParams p, int s0, int n_rows, int TM, int TN, int splits) {
  using G = LmGemmOf<SMALL, true>;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int tm, tn, split;
  if (!lm_tile<G>(blockIdx.x, TM, TN, splits, tm, tn, split)) return;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;
  const int m0 = tm * G::BM, n0 = tn * G::BN, nk_all = (p.vocab + kLmBK - 1) / kLmBK;
  const int kt0 = (int)((int64_t)nk_all * split / splits), nk = (int)((int64_t)nk_all * (split + 1) / splits) - kt0;
  const int word0 = kt0 * kLmBK;
  typename G::OpA a;
  typename G::OpB b;
  a.init(p.dlogits + word0, p.v_pad, p.tile_tokens, m0, nk, wave, lane);
  b.init(p.w + (int64_t)word0 * p.ld_w, p.ld_w, p.vocab - word0, n0, nk, wave, lane);
  G gemm;
  gemm.run(smem, a, b, nk, wm, wn, wave, lane);   // dLogits is zero beyond the vocabulary
  const bool partial = splits > 1;
  float* out_f32 = partial ? p.logits + (int64_t)split * TM * G::BM * p.d_model : (float*)p.dh + (int64_t)s0 * p.ld_dh;
  const int64_t ld = partial ? p.d_model : p.ld_dh;
#pragma unroll
  for (int half = 0; half < G::HALVES; ++half)
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + 128 * half + wm * 64 + 16 * mb + 4 * g + v;
        if (row >= n_rows) continue;
        const int64_t off = row * ld + n0 + wn * 64 + r;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
          const float x = gemm.acc[half][mb][nb][v];
          if (partial || p.dh_is_f32) out_f32[off + 16 * nb] = x;
          else ((__bf16*)p.dh)[(int64_t)s0 * p.ld_dh + off + 16 * nb] = (__bf16)x;
        }
      }
}

// dH rows from the partial sums of a split contraction: one work-item per eight columns.  stride: elements per part.
__global__ __launch_bounds__(256) void lm_dh_sum_kernel(LmHeadParams p, int s0, int n_rows, int splits, int64_t stride) {
  const int d8 = p.d_model / 8;
  const int64_t i = blockIdx.x * 256ll + threadIdx.x;
  if (i >= (int64_t)n_rows * d8) return;
  const int64_t row = i / d8, col = (i - row * d8) * 8;
  const float* src = p.logits + row * p.d_model + col;
  f32x4 x0 = *reinterpret_cast<const f32x4*>(src), x1 = *reinterpret_cast<const f32x4*>(src + 4);
  for (int s = 1; s < splits; ++s) {
    x0 += *reinterpret_cast<const f32x4*>(src + s * stride);
    x1 += *reinterpret_cast<const f32x4*>(src + s * stride + 4);
  }
  const int64_t off = (s0 + row) * p.ld_dh + col;
  if (p.dh_is_f32) {
    *reinterpret_cast<f32x4*>((float*)p.dh + off) = x0;
    *reinterpret_cast<f32x4*>((float*)p.dh + off + 4) = x1;
  } else {
    const bf16x8 y = {(__bf16)x0[0], (__bf16)x0[1], (__bf16)x0[2], (__bf16)x0[3],
                      (__bf16)x1[0], (__bf16)x1[1], (__bf16)x1[2], (__bf16)x1[3]};
    *reinterpret_cast<bf16x8*>((__bf16*)p.dh + off) = y;
  }
}

// ---------------------------------------------------------------------------------------------
// 4. dW (+)= dLogits^T H_i, computed as its transpose dW^T = H_i^T dLogits (rows: hidden,
//    columns: words, contraction: tokens of the tile).  Both factors are stored with the token as
//    the row, and an operand read column-wise costs twice the LDS instructions of a row-wise one;
//    A, of which a wave reads eight operands per k-step (four per phase), is therefore taken from a
//    transposed copy of H_i (a few MB, written by lm_transpose_h_kernel once per sequence tile), and only
//    B (dLogits), four operands per k-step that stay in registers for both phases, uses the transposing
//    read.  A lane then owns a word: it adds four consecutive hidden columns of that word's row of dW at a time.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void lm_transpose_h_kernel(LmHeadParams p, int s0, int n_rows) {
  __shared__ __bf16 tile[64][66];
  const int t0 = blockIdx.x * 64, d0 = blockIdx.y * 64, tid = threadIdx.x;   // 64 tokens x 64 hidden columns
  for (int i = tid; i < 64 * 8; i += 256) {
    const int tok = i >> 3, c8 = (i & 7) * 8;
    bf16x8 x = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
    if (t0 + tok < n_rows) x = *reinterpret_cast<const bf16x8*>(p.h + (int64_t)(s0 + t0 + tok) * p.ld_h + d0 + c8);
#pragma unroll
    for (int e = 0; e < 8; ++e) tile[tok][c8 + e] = x[e];
  }
  __syncthreads();
  for (int i = tid; i < 64 * 8; i += 256) {
    const int dc = i >> 3, t8 = (i & 7) * 8;
    bf16x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = tile[t8 + e][dc];
    *reinterpret_cast<bf16x8*>(p.ht + (int64_t)(d0 + dc) * p.tile_tokens + t0 + t8) = x;
  }
}

template <bool SMALL>
__global__ __launch_bounds__((LmGemmOf<SMALL, true>::THREADS), 2) void lm_dw_kernel(LmHeadParams p, int s0, int n_rows, int TM, int TN, int accumulate) {
  using G = LmGemmOf<SMALL, true>;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int tm, tn, split;
  if (!lm_tile<G>(blockIdx.x, TM, TN, 1, tm, tn, split)) return;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;
  const int m0 = tm * G::BM, n0 = tn * G::BN, nk = (n_rows + kLmBK - 1) / kLmBK;      // m0: hidden column, n0: word
  typename G::OpA a;
  typename G::OpB b;
  a.init(p.ht, p.tile_tokens, p.d_model, m0, nk, wave, lane);
  b.init(p.dlogits, p.v_pad, p.tile_tokens, n0, nk, wave, lane);
  G gemm;
  gemm.run(smem, a, b, nk, wm, wn, wave, lane);    // both factors are zero beyond n_rows
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) {
    const int word = n0 + wn * 64 + 16 * nb + r;
    if (word >= p.vocab) continue;
    float* dst = p.dw + (int64_t)word * p.ld_dw + m0 + wm * 64 + 4 * g;
    f32x4 old[G::HALVES][4];
#pragma unroll
    for (int i = 0; i < 4 * G::HALVES; ++i) old[i / 4][i % 4] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (accumulate) {   // all loads before the first store
#pragma unroll
      for (int i = 0; i < 4 * G::HALVES; ++i) old[i / 4][i % 4] = *reinterpret_cast<const f32x4*>(dst + 128 * (i / 4) + 16 * (i % 4));
    }
#pragma unroll
    for (int i = 0; i < 4 * G::HALVES; ++i) *reinterpret_cast<f32x4*>(dst + 128 * (i / 4) + 16 * (i % 4)) = gemm.acc[i / 4][i % 4][nb] + old[i / 4][i % 4];
  }
}

__global__ __launch_bounds__(256) void lm_zero_dw_kernel(LmHeadParams p) {
  const int d4 = p.d_model / 4;
  const int64_t total = (int64_t)p.vocab * d4;
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256)
    *reinterpret_cast<f32x4*>(p.dw + (i / d4) * p.ld_dw + (i % d4) * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
}

}  // namespace

int64_t lm_head_workspace_bytes(int64_t tile_tokens, int64_t vocab, int64_t d_model) {
  const int64_t v_pad = (vocab + 255) / 256 * 256;
  return tile_tokens * v_pad * 4 + tile_tokens * v_pad * 2 + (v_pad / 128) * tile_tokens * 8 + d_model * tile_tokens * 2;
}

void lm_head_tile_plan(const LmHeadParams& p, int32_t out[6]) {
  const int n_rows = std::min(p.n_tokens, p.tile_tokens);
  const LmPlan plans[3] = {lm_plan_logits(p, n_rows), lm_plan_dh(p, n_rows), lm_plan_dw(p, n_rows)};
  for (int i = 0; i < 3; ++i) {
    out[2 * i] = plans[i].tile();
    out[2 * i + 1] = plans[i].splits;
  }
}

hipError_t launch_lm_head_loss(const LmHeadParams& p, hipStream_t stream) {
  const int want_grad = (p.dh || p.dw) ? 1 : 0;
  if (p.n_tokens == 0 && p.dw && !p.acc_dw) {
    hipLaunchKernelGGL(lm_zero_dw_kernel, dim3(2048), dim3(256), 0, stream, p);
    return hipGetLastError();
  }
  for (int s0 = 0; s0 < p.n_tokens; s0 += p.tile_tokens) {
    const int n_rows = p.n_tokens - s0 < p.tile_tokens ? p.n_tokens - s0 : p.tile_tokens;
    auto launch = [&](const LmPlan& g, auto* big, auto* small, int last) {
      const dim3 grid(lm_grid(g.TM, g.TN, g.splits, g.small));
      if (g.small) hipLaunchKernelGGL(small, grid, dim3(LmGemmSmall<true>::THREADS), LmGemmSmall<true>::LDS, stream, p, s0, n_rows, g.TM, g.TN, last);
      else hipLaunchKernelGGL(big, grid, dim3(kLmThreads), LmGemm<true>::LDS, stream, p, s0, n_rows, g.TM, g.TN, last);
    };
    const int k_rows = (n_rows + 63) / 64 * 64;
    const LmPlan logits = lm_plan_logits(p, n_rows), dh = lm_plan_dh(p, n_rows), dw = lm_plan_dw(p, n_rows);
    launch(logits, lm_logits_kernel<false>, lm_logits_kernel<true>, logits.splits);
    const dim3 loss_grid(want_grad ? k_rows : n_rows);
    if (logits.splits > 1)
      hipLaunchKernelGGL((lm_loss_dlogits_kernel<true>), loss_grid, dim3(lm_loss_threads(true)), 0, stream, p, s0, n_rows, want_grad, 0, logits.splits,
                         logits.TN * logits.tile());
    else
      hipLaunchKernelGGL((lm_loss_dlogits_kernel<false>), loss_grid, dim3(lm_loss_threads(false)), 0, stream, p, s0, n_rows, want_grad,
                         (p.vocab + 127) / 128, 1, 0);
    if (p.dh) {
      launch(dh, lm_dh_kernel<false>, lm_dh_kernel<true>, dh.splits);
      if (dh.splits > 1)
        hipLaunchKernelGGL(lm_dh_sum_kernel, dim3((uint32_t)(((int64_t)n_rows * (p.d_model / 8) + 255) / 256)), dim3(256), 0, stream,
                           p, s0, n_rows, dh.splits, (int64_t)dh.TM * dh.tile() * p.d_model);
    }
    if (p.dw) {
      hipLaunchKernelGGL(lm_transpose_h_kernel, dim3(k_rows / 64, p.d_model / 64), dim3(256), 0, stream, p, s0, n_rows);
      launch(dw, lm_dw_kernel<false>, lm_dw_kernel<true>, (p.acc_dw || s0 > 0) ? 1 : 0);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace burst
