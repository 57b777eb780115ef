// Backward step kernels (Alg. 2, with the softmax scale restored):
//   S = scale Q K^T; P = exp(S - Lse); dV += P^T dO; dP = dO V^T; dS = P o (dP - D);
//   dK += scale dS^T Q; dQ += scale dS K.
//
// Two kernels, each owning its outputs outright (no atomics, results are run-to-run identical); a short step launches
// the work-groups of both together (step_bwd_both_kernel):
//
//  * dQ kernel, query-stationary, the forward kernel's structure (16x16x32 MFMAs, direct LDS loads, the two waves of
//    a SIMD taking matrix and vector phases in turn): S^T = K Q^T and dP^T = V dO^T come out with the key index
//    in the accumulator registers, dS^T is packed to bf16 in place and fed back as the B operand of
//    dQ^T = K^T dS^T, whose A operand is the K tile read column-wise (transposing LDS reads) from the same LDS
//    copy that served S^T row-wise.  Bound by the matrix pipe under the chip's power limit: 96 MFMAs of 16 clocks
//    per tile and wave against about 900 clocks of vector work, which the other wave's matrix phase hides.
//    128K-token ring backward (dQ and dK/dV): 56.3 -> 52.6 ms against the 32x32x16 kernel with register staging.
//
//  * dK/dV kernel, key-stationary: a lane owns two key rows; K and V rows live in registers as B
//    operands, S = Q K^T and dP = dO V^T come out with the query index in the accumulator registers,
//    P and dS are packed in place and fed back as B operands of dV^T = dO^T P and dK^T = Q^T dS,
//    whose A operands are the dO and Q tiles read column-wise from the LDS copies that served
//    S and dP row-wise.  With grouped-query attention the work-group walks the query heads of its
//    group, so dK and dV are summed over the group in registers.
//
// At d = 64 the vector unit is what dQ needs most (75 % busy, matrix pipe 60 %; 32 heads x 16384 rows), and it is filled by waves that keep no common
// rhythm (fwd.hip); dK/dV needs both alike (57 and 58 %) and waits for LDS.  The dQ kernel runs four
// waves a work-group, three work-groups a CU, 32 key rows after the other (144-150 registers); dK/dV, whose P-waves and dS-waves need
// their rhythm, and the joint launch run two work-groups of eight waves a CU in 128 registers, with tiles asked for two ahead so that
// three are in LDS, where the launch has more than one work-group for each CU and, joint, enough work (crowded).  us, one work-group a CU
// and so: dQ 4 x 12 heads x 1500 rows 77, 57; 4 x 64/8 x 1879, window 504, three steps 232, 160; 1 x 20000 380, 292; 32 x 16384
// 1412, 1393; 12 x 24749 2520, 2570; dK/dV 4 x 12 x 1500 90, 79; 32 x 3010, batch 2, window 1219 152, 122; 32 x 16384 1930, 1812; 12 x 24749
// 3590, 3470; 64/16 x 8548 causal 2290, 2330.  (A dK/dV kernel without roles, a wave with K, V and both sums: two work-groups of four
// waves a CU, 196 registers, 32 x 16384 2065; with 16 keys a wave, three work-groups, 2380.)
#include "common.hpp"
#include "kernels.hpp"
#include "mfma16.hpp"

namespace burst {

template <int D>
constexpr int kDqWaves = D == 128 ? 8 : 4;       // of the dQ kernel: two per SIMD that take turns; three work-groups per CU (fwd.hip)
// tiles of both streamed operands in LDS.  TURNS: one work-group has the CU and its waves take turns; else several share it
template <bool TURNS>
constexpr int kBwdSlots = TURNS ? 4 : 3;

// lse in log2 units, with -inf mapped to +inf so that exp2(x - lse2) = 0 for a dead row
__device__ __forceinline__ float lse_to_log2(float lse) { return lse == -INFINITY ? INFINITY : lse * kLog2e; }

// ---------------------------------------------------------------------------------------------
template <int D, int NW, bool BLK, bool MULTI, int AHEAD, bool TURNS>   // BLK: with a block-wise sparse mask; MULTI: more than one step
__device__ __forceinline__ void dq_block(const BwdParams& p, char* smem, int block) {   // smem: [SLOTS][K tile, V tile], open flags
  constexpr int BK = 64, MB = BK / 16, NB = 2, DK = D / 32, DB = D / 16, BQ = 32 * NW, NT = 64 * NW;
  constexpr int TILE = BK * 2 * D, SLOTS = kBwdSlots<TURNS>;

  const int group = p.q_heads / p.kv_heads;
  const BlockMap bm = map_block<true>(block, p.batch * p.kv_heads, group, p.q_runs.total(), p.q_side_by_side);
  if (!bm.valid) return;
  const int b = __builtin_amdgcn_readfirstlane(bm.key / p.kv_heads), hk = bm.key - b * p.kv_heads, hq = hk * group + bm.head_in_group;

  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: everything derived from it stays wave-uniform
  const int sq = p.sq, n_steps = MULTI ? p.n_steps : 1;
  const MaskDev q_side = p.step[0].mask;   // all steps have the same
  const int q_blk0 = p.q_runs.tile_of(bm.tile) * BQ, q_blk1 = min(q_blk0 + BQ, sq);
  const int q_w0 = q_blk0 + wave * 32, q_w1 = min(q_w0 + 32, sq);

  // Q and dO as B operands: lane holds rows q_w0 + 16 nb + r, columns 32 ks + 8g .. +7
  bf16x8 qreg[DK][NB], doreg[DK][NB];
  int q_pos[NB], klo[NB], khi[NB];   // positions of the lane's query rows, the key rows they see of a step
  float lse2[NB], dval[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = min(q_w0 + 16 * nb + r, sq - 1);
    q_pos[nb] = axis_position(axis_of<true>(q_side), row);
    const __bf16* qs = (const __bf16*)p.q.ptr + b * p.q.sb + hq * p.q.sh + (int64_t)row * p.q.ss + 8 * g;
    const __bf16* gs = (const __bf16*)p.d_o.ptr + b * p.d_o.sb + hq * p.d_o.sh + (int64_t)row * p.d_o.ss + 8 * g;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      qreg[ks][nb] = *reinterpret_cast<const bf16x8*>(qs + ks * 32);
      doreg[ks][nb] = *reinterpret_cast<const bf16x8*>(gs + ks * 32);
    }
    lse2[nb] = lse_to_log2(p.lse.ptr[b * p.lse.sb + hq * p.lse.sh + row]);
    dval[nb] = p.d.ptr[b * p.d.sb + hq * p.d.sh + row];
  }
  const float c = p.scale * kLog2e;

  f32x4 dq[DB][NB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) dq[db][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Positions of the work-group's and the wave's query rows
  int qlo_blk, qhi_blk, qlo_w = 0, qhi_w = 0;
  range_minmax<true>(q_side, q_blk0, q_blk1, qlo_blk, qhi_blk);
  if (q_w0 < q_w1) range_minmax<true>(q_side, q_w0, q_w1, qlo_w, qhi_w);

  // Open flags of the key tiles against this work-group's query block (block-wise sparse mask)
  uint8_t* open_flags = nullptr;
  if (BLK) {
    open_flags = reinterpret_cast<uint8_t*>(smem + SLOTS * 2 * TILE);
    fill_open_flags<true, BK>(q_side, open_flags, q_blk0, p.step[0].sk, tid, NT);
    __syncthreads();
  }
  OperandAddr<D> ad;
  ad.init(lane);
  TileRanges tiles;   // class of a step's key tiles against this wave's 32 query rows
  bool windowed;
  uint32_t lds0 = (uint32_t)(uintptr_t)(lds_bytes)smem;

  // The two waves of a SIMD take a tile's matrix phase and its vector phase in turn, as in the forward kernel:
  // waves 4-7 run one barrier behind waves 0-3.  Iteration t, tile t in slot t mod 4:
  //   matrix phase: dQ += K(t)^T dS(t), then S(t+1) = K Q^T and dP(t+1) = V dO^T
  //   vector phase: dS(t+1)
  // A barrier ends every phase.  Tile t+3 is asked for in the matrix phase of iteration t (its slot held tile
  // t-1, which the later half finished a barrier ago).  At the end of that phase a wave waits for its share of tile
  // t+2, so that both halves' shares are there a barrier before either half's products of iteration t+1 read it.
  // Before and behind the run of tiles of which its rows see something a wave only asks for loads and meets the others,
  // as in the forward kernel.
  auto k_lds = [&](int s_) { return lds0 + s_ * 2 * TILE; };
  auto v_lds = [&](int s_) { return lds0 + s_ * 2 * TILE + TILE; };
  constexpr int LOADS = KvStream<D, BK, NW, BLK, false>::LOADS, NL = KvStream<D, BK, NW, BLK, false>::N;
  // The steps one after the other; dQ stays in registers
#pragma clang loop unroll(disable)
  for (int step = 0; step < n_steps; ++step) {
    const BwdStep& st = p.step[MULTI ? step : 0];
    const MaskDev mk = st.mask;
    const int sk = st.sk;
    windowed = mk.window != kNoWindow;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) visible_rows<true>(mk, q_pos[nb], sk, klo[nb], khi[nb]);
    tiles.init(row_intervals<false>(mk, qlo_w, qhi_w, sk, q_w0 >= q_w1), sk, BK);
    KvStream<D, BK, NW, BLK, false> walk;
    walk.init(mk, st.k, st.v, b, hk, sk, qlo_blk, qhi_blk, wave, lane, open_flags);
    wait_global_loads();
    if (step > 0) __syncthreads();   // the later half may still read the last tile of the step before
    pin(lds0);   // (LDS addresses worked out once for all steps would cost the registers)
    bf16x8 ds[MB / 2][NB];
    // dS of 32 key rows for the query rows nb from their scores and dP
    auto d_scores32 = [&](int nb, f32x4& x, f32x4& y, const f32x4& dpx, const f32x4& dpy) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        x[v] = __builtin_amdgcn_exp2f(c * x[v] - lse2[nb]) * (dpx[v] - dval[nb]);
        y[v] = __builtin_amdgcn_exp2f(c * y[v] - lse2[nb]) * (dpy[v] - dval[nb]);
      }
      return pack_pair(x, y);
    };
    // dS of the tile at key row k0_, of which the wave sees something, for the query rows nb: from their scores and dP
    auto d_scores = [&](int k0_, int nb, auto&& score, auto&& d_p) {   // score(mb), d_p(mb): f32x4
      if (!tiles.full(k0_)) {
#pragma unroll
        for (int half = 0; half < MB / 2; ++half)
          mask_rows32(score(2 * half), score(2 * half + 1), k0_ + 32 * half, g, klo[nb], khi[nb], windowed);
      }
#pragma unroll
      for (int ch = 0; ch < MB / 2; ++ch) ds[ch][nb] = d_scores32(nb, score(2 * ch), score(2 * ch + 1), d_p(2 * ch), d_p(2 * ch + 1));
    };
    if (!TURNS) {   // tile t in slot t mod 3: products and vector work one after the other, a barrier for each tile
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
            bf16x8 first[AHEAD];
#pragma unroll
            for (int half = 0; half < 2; ++half) {   // 32 key rows after the other: registers
              constexpr int HALF = 32 * 2 * D, NP = NW == 8 ? 1 : NB;   // (eight waves: and 16 query rows after the other)
              const uint32_t kh = k_lds(slot) + half * HALF, vh = v_lds(slot) + half * HALF;
#pragma unroll
              for (int n0 = 0; n0 < NB; n0 += NP) {
                f32x4 s[2][NP], dp[2][NP];
                bf16x8 qp[DK][NP], dop[DK][NP];
#pragma unroll
                for (int i = 0; i < DK * NP; ++i) {
                  qp[i / NP][i % NP] = qreg[i / NP][n0 + i % NP];
                  dop[i / NP][i % NP] = doreg[i / NP][n0 + i % NP];
                }
                rows_fetch<D, 2, AHEAD>(kh, ad, 0, first);
                rows_product_pair<D, 2, NP, AHEAD>(kh, vh, ad, qp, dop, s, dp, first);
#pragma unroll
                for (int nb = n0; nb < n0 + NP; ++nb) {
                  f32x4 &x = s[0][nb - n0], &y = s[1][nb - n0];
                  if (!tiles.full(kb)) mask_rows32(x, y, kb + 32 * half, g, klo[nb], khi[nb], windowed);
                  ds[half][nb] = d_scores32(nb, x, y, dp[0][nb - n0], dp[1][nb - n0]);
                }
              }
            }
            cols_fetch<D, AHEAD>(k_lds(slot), ad, 0, first);
            cols_product<D, MB / 2, NB, AHEAD>(k_lds(slot), ad, 0, ds, dq, first);
          }
          kb = kc;
          kc = kn;
          slot = slot == 2 ? 0 : slot + 1;
          pin(kb, kc, slot);
        } while (kb >= 0);
        wait_global_loads();             // tiles past the end of the walk
      }
    } else if (walk.valid()) {
      int kb = walk.k0;   // iteration t: kb, kc are the first rows of tiles t+1, t+2
      walk.issue(k_lds(0), v_lds(0), wave, lane);
      int kc = walk.cursor();
      walk.issue(k_lds(1), v_lds(1), wave, lane);
      int kn = walk.cursor();
      walk.issue(k_lds(2), v_lds(2), wave, lane);
      wait_loads_barrier<2 * LOADS>();              // tile 0
      if (wave >= NW / 2) phase_barrier();
      int slot = 3;
      bool live;
      bf16x8 first[AHEAD];
      // The first tile of several steps at d = 128: dQ of the steps before, both products of 32 query rows and their operands do
      // not fit the registers, so the rows go 16 after the other, each through its vector work (elsewhere that would be one
      // vector phase more before the later half's first products, 0.5 us of a step)
      constexpr bool WHOLE = !(MULTI && D == 128);
      any_value(ds);
      any_value(first);
      for (;;) {   // iterations -1 .., up to the wave's first tile
        const int slot1 = (slot + 1) & 3;
        live = tiles.some(kb);
        f32x4 s[MB][NB], dp[MB][NB];
        auto scores = [&]() {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            d_scores(kb, nb, [&](int mb) -> f32x4& { return s[mb][nb]; }, [&](int mb) -> f32x4& { return dp[mb][nb]; });
        };
        if (live && WHOLE) {
          rows_fetch<D, MB, AHEAD>(k_lds(slot1), ad, 0, first);
          rows_product_pair<D, MB, NB, AHEAD>(k_lds(slot1), v_lds(slot1), ad, qreg, doreg, s, dp, first);
        } else if (live) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            f32x4 s1[MB][1], dp1[MB][1];
            bf16x8 q1[DK][1], do1[DK][1], ahead[2];
#pragma unroll
            for (int ks = 0; ks < DK; ++ks) {
              q1[ks][0] = qreg[ks][nb];
              do1[ks][0] = doreg[ks][nb];
            }
            rows_fetch<D, MB, 2>(k_lds(slot1), ad, 0, ahead);
            rows_product_pair<D, MB, 1, 2>(k_lds(slot1), v_lds(slot1), ad, q1, do1, s1, dp1, ahead);
            d_scores(kb, nb, [&](int mb) -> f32x4& { return s1[mb][0]; }, [&](int mb) -> f32x4& { return dp1[mb][0]; });
          }
        }
        wait_loads_barrier<LOADS>();                // tile t+2
        slot = slot1;
        if (live) {
          if (WHOLE) scores();
          cols_fetch<D, AHEAD>(k_lds(slot), ad, 0, first);
        }
        phase_barrier();
        kb = kc;
        kc = kn;
        if (live || kb < 0) break;
        kn = walk.cursor();
        walk.issue(k_lds((slot + 3) & 3), v_lds((slot + 3) & 3), wave, lane);
      }
      if (live) {
        uint32_t kt = k_lds(slot), k1 = k_lds((slot + 1) & 3), v1 = v_lds((slot + 1) & 3);   // slot t mod 4 and the next
        uint32_t kl = k_lds((slot + 3) & 3), vl = v_lds((slot + 3) & 3);
        kn = walk.cursor();
        walk.begin(wave, lane);
        for (;;) {
          // ---- matrix phase; everything else that an iteration computes stands behind its MFMAs or in the vector phase
          f32x4 s[MB][NB], dp[MB][NB];
          bf16x8 first_rows[AHEAD];
          constexpr int NCOLS = MB / 2 * DB;
          cols_product<D, MB / 2, NB, AHEAD>(kt, ad, 0, ds, dq, first, [&](int i) {
            if (i < NL) walk.load_v(i, vl, wave);
            if (i >= NL && i < 2 * NL) walk.load_k(i - NL, kl, wave);
            if (i >= 2 * NL && i < 2 * NL + walk.PARTS) walk.end(i - 2 * NL);
            if (i >= NCOLS - AHEAD) {
              const int f = i - (NCOLS - AHEAD);
              first_rows[f] = rows_operand<D>(k1, ad, 16 * (f % MB), f / MB);
            }
          });
          if (tiles.behind(kb)) break;
          rows_product_pair<D, MB, NB, AHEAD>(k1, v1, ad, qreg, doreg, s, dp, first_rows);
          wait_loads_barrier<LOADS>();              // tile t+2
          // ---- vector phase
          const int tile_k0 = kb;
          slot = (slot + 1) & 3;
          vl = kt + TILE;   // (the slot before)
          kl = kt;
          kt = k1;
          k1 = k_lds((slot + 1) & 3);
          v1 = k1 + TILE;
          kb = kc;
          kc = kn;
          kn = walk.cursor();
          walk.begin(wave, lane);
          pin(slot, kt, k1, v1, kl, vl, kb, kc, kn);
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            d_scores(tile_k0, nb, [&](int mb) -> f32x4& { return s[mb][nb]; }, [&](int mb) -> f32x4& { return dp[mb][nb]; });
          cols_fetch<D, AHEAD>(kt, ad, 0, first);
          phase_barrier();
        }
      }
      while (kb >= 0) {   // the rest of the walk is the other waves'
        wait_loads_barrier<LOADS>();
        slot = (slot + 1) & 3;
        phase_barrier();
        kb = kc;
        kc = kn;
        kn = walk.cursor();
        walk.issue(k_lds((slot + 3) & 3), v_lds((slot + 3) & 3), wave, lane);
      }
      wait_global_loads();   // tiles past the end of the walk
      if (wave < NW / 2) phase_barrier();
    }
  }

#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = q_w0 + 16 * nb + r;
    if (row >= sq) continue;
    float* dst = (float*)p.dq.ptr + b * p.dq.sb + (int64_t)row * p.dq.ss + hq * p.dq.sh + 4 * g;
    f32x4 old[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) old[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (p.acc_dq) {   // all loads before the first store
#pragma unroll
      for (int db = 0; db < DB; ++db) old[db] = *reinterpret_cast<const f32x4*>(dst + 16 * db);
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(dst + 16 * db) = dq[db][nb] * p.scale + old[db];
  }
}

// ---------------------------------------------------------------------------------------------
// dK/dV kernel.  Eight waves per work-group, two per SIMD, in two roles that share each block of 32 key rows:
//   P-wave  (waves 0-3): K rows in registers; S = Q K^T, P = exp2(..) -> bf16, handed over through LDS,
//                        dV^T += dO^T P.
//   dS-wave (waves 4-7): V rows in registers; dP = dO V^T - D, dS = P o dP, dK^T += Q^T dS.
// Each role carries one 32 x D accumulator and one stationary operand, which is what lets two waves fit on a
// SIMD; the two roles are separate instruction streams.  A wave's work on a query tile (64 rows) is a matrix phase
// and a vector phase, a barrier ends every phase, and the dS-waves run one phase behind, so that the two waves of a
// SIMD hand the matrix pipe to each other.  Iteration t:
//   P-wave:  matrix: dV^T += dO(t)^T P(t), then S(t+1) from Q(t+1) and -lse      vector: P(t+1), stored to LDS
//   dS-wave: matrix: dK^T -= Q(t)^T dS(t), then D - dP(t+1) from dO(t+1) and D   vector: -dS(t+1) from P(t+1)
// (With three tiles in LDS, at d = 64: tile t+2 is asked for while P-waves run the matrix phase of iteration t, by both roles; it is
// there when the dS-waves have run theirs, and P-waves bring lse into its form at the head of the matrix phase that needs it.)
// P(t+1) is stored in the phase before the one that reads it and read a phase before P(t+2) is stored: one copy.
// Tile t+3 is asked for in the matrix phase of iteration t, into the slot (of four) of tile t-1, which the dS-waves
// left a barrier ago; a wave waits for its share of tile t+2 at the end of that phase, two barriers before either
// role's products read it.  lse or D rows come with a tile into the wave's own LDS, raw; the P-wave brings its rows into the
// form the accumulators start from in the vector phase before, the dS-wave starts from D as it is.
// What bounds it: one wave alone on the matrix pipe, and what a phase costs beside its MFMAs.  A wave issues an MFMA of 16 clocks
// every 18.4 at best, every 20-21 with an operand read for every two (probe); between two barriers lie 1520 (P) and 1870 (dS) clocks of
// 64 MFMAs while the other role's vector phase, whose instructions take 9 clocks beside MFMAs and its exponentials 15-18, runs
// for 1460 and 980 (shader clock read at the barriers).  So what stood between the barriers and was neither went: the walk's
// scalar arithmetic stands behind MFMAs (pin), P is read in one LDS round trip instead of four, the dS-wave needs none for
// D, the barrier waits for the stores of P and not for the operand prefetch behind them, a direct load waits one state for
// m0 instead of four.  16384 x 16384 rows, 32 heads, d = 128: 3605 -> 3377 us a step; 8192 rows, d = 64: 621 -> 518.
// 128K-token ring backward 52.6 -> 48.7 ms against 32x32x16 MFMAs with tiles staged through registers by the P-waves
// and the vector work sliced behind each wave's own MFMAs; d = 64, 1500 rows, 4 x 12 heads: 120 -> 95 us per step.
template <int D, bool TURNS>
struct DkdvLds {
  static constexpr int BQ = 64, SLOTS = kBwdSlots<TURNS>, TILE = BQ * 2 * D;
  static constexpr int Q_OFF = 0, DO_OFF = SLOTS * TILE;
  static constexpr int ROW_OFF = DO_OFF + SLOTS * TILE, ROW = BQ * 4;   // [wave][slot]
  static constexpr int P_OFF = ROW_OFF + 8 * SLOTS * ROW, P_PAIR = BQ * 32 * 2;   // [pair][chunk, key block][lane]
  static constexpr int BYTES = P_OFF + 4 * P_PAIR;
};

// BKV = 128: the four pairs own 32 key rows each and run through all 64 rows of a query tile.  BKV = 64, for launches
// with too few key tiles to fill the CUs: two pairs share 32 key rows, each runs through 32 of the 64 query rows (the
// same operand reads per MFMA, half the MFMAs per phase), and the second one's sums are added through LDS at the end.
template <int D, int ROLE, bool BLK, int BKV, bool TURNS>
__device__ __forceinline__ void dkdv_role(const BwdParams& p, const BwdStep& st, char* smem, int b, int hk, int kv_tile, int wave) {
  constexpr int BQ = 64, QS = 128 / BKV, ROWS = BQ / QS, MB = ROWS / 16, NB = 2, DK = D / 32, DB = D / 16, NW = 8, AHEAD = TURNS ? kAhead16 : 3;
  using L = DkdvLds<D, TURNS>;
  constexpr int SLOTS = L::SLOTS;
  constexpr bool NEAR = !TURNS;   // a tile is asked for two tiles ahead, not three

  const int group = p.q_heads / p.kv_heads;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4, pair = wave & 3;
  const int sq = p.sq, sk = st.sk;
  const MaskDev mk = st.mask;
  const int k_blk0 = st.k_runs.tile_of(kv_tile) * BKV, k_blk1 = min(k_blk0 + BKV, sk);
  const int k_w0 = k_blk0 + (QS == 1 ? pair : pair & 1) * 32, k_w1 = min(k_w0 + 32, sk);
  const int row0 = QS == 1 ? 0 : (pair >> 1) * ROWS;   // first row of the wave's part of a query tile
  const float c = p.scale * kLog2e;

  // K rows (P-wave) or V rows (dS-wave) as the B operand: lane holds rows k_w0 + 16 nb + r, columns 32 ks + 8g .. +7
  bf16x8 xreg[DK][NB];
  int qlo[NB], qhi[NB];   // query rows that see the lane's key rows (P-wave)
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = min(k_w0 + 16 * nb + r, sk - 1);
    if (ROLE == 0) visible_rows<false>(mk, axis_position(axis_of<false>(mk), row), sq, qlo[nb], qhi[nb]);
    const TensorDev& src = ROLE == 0 ? st.k : st.v;
    const __bf16* x = (const __bf16*)src.ptr + b * src.sb + hk * src.sh + (int64_t)row * src.ss + 8 * g;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      xreg[ks][nb] = *reinterpret_cast<const bf16x8*>(x + ks * 32);
      // K rows carry the factor scale * log2(e) (rounded to bf16 once per work-group) and the S accumulators start
      // from -lse: P = exp2 of the accumulator, no per-score multiply-add.  The extra rounding of K moves P by a
      // few 1e-3 relative, the size of the bf16 rounding P undergoes anyway before the dV product (the paper
      // fixes no precision); only this kernel does it: the forward kernel's Lse is held to 1e-3 absolute and
      // keeps the exact multiply-add.
      // V rows change their sign, which is exact: the dP accumulators then start from D as it comes, and dS and dK^T carry
      // the sign until the results are written.
#pragma unroll
      for (int e = 0; e < 8; ++e) xreg[ks][nb][e] = ROLE == 0 ? (__bf16)((float)xreg[ks][nb][e] * c) : -xreg[ks][nb][e];
    }
  }

  f32x4 acc[DB][NB];   // dV^T (P-wave) or dK^T (dS-wave)
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[db][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

  int klo_blk, khi_blk, klo_w = 0, khi_w = 0;
  range_minmax<false>(mk, k_blk0, k_blk1, klo_blk, khi_blk);
  if (k_w0 < k_w1) range_minmax<false>(mk, k_w0, k_w1, klo_w, khi_w);
  TileRanges tiles;
  tiles.init(row_intervals<true>(mk, klo_w, khi_w, sq, k_w0 >= k_w1), sq, ROWS);

  uint8_t* open_flags = nullptr;
  if (BLK) {
    open_flags = reinterpret_cast<uint8_t*>(smem + L::BYTES);
    if (ROLE == 0) fill_open_flags<false, BQ>(mk, open_flags, k_blk0, sq, tid, 256);
    __syncthreads();
  }
  OperandAddr<D> ad;
  ad.init(lane);
  QStream<D, BQ, NW, BLK> walk;
  walk.init(p.q, p.d_o, ROLE == 0 ? p.lse : p.d, b, hk * group, group, visible_tiles<true, BQ>(mk, klo_blk, khi_blk, sq), sq, wave,
            lane, open_flags);
  wait_global_loads();
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_bytes)smem;
  auto q_lds = [&](int s_) { return lds0 + L::Q_OFF + s_ * L::TILE; };
  auto o_lds = [&](int s_) { return lds0 + L::DO_OFF + s_ * L::TILE; };
  auto row_off = [&](int s_) { return L::ROW_OFF + (wave * L::SLOTS + s_) * L::ROW; };
  auto after = [](int s_) { return SLOTS == 4 ? (s_ + 1) & 3 : s_ == 2 ? 0 : s_ + 1; };
  // the wave's rows of the tile of the product that starts from a row vector, and of the product that fills acc
  auto rows_lds = [&](int s_) { return (ROLE == 0 ? q_lds(s_) : o_lds(s_)) + row0 * 2 * D; };
  auto cols_lds = [&](int s_) { return (ROLE == 0 ? o_lds(s_) : q_lds(s_)) + row0 * 2 * D; };
  bf16x8* const hand = reinterpret_cast<bf16x8*>(smem + L::P_OFF + pair * L::P_PAIR) + lane;
  constexpr int LOADS = QStream<D, BQ, NW, BLK>::LOADS;

  f32x4 s[MB][NB], init[MB];   // S - lse2 or D - dP of a tile; -lse2 or D of the lane's rows of it
  bf16x8 ps[MB / 2][NB];       // P or -dS
  auto issue = [&](int s_) {
    walk.begin(wave, lane);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) walk.load(i, q_lds(s_), o_lds(s_), lds0 + row_off(s_), wave);
    walk.advance();
  };
  // P-wave: lse of a slot's rows -> accumulator start, in place (a dead row's lse of -inf gives P = 0)
  auto raw_rows = [&](int s_) { return reinterpret_cast<float*>(smem + row_off(s_)) + lane; };
  auto init_rows = [&](int s_, int mb) { init[mb] = *reinterpret_cast<const f32x4*>(smem + row_off(s_) + 4 * (row0 + 16 * mb + 4 * g)); };
  // The vector phase, of the tile at query row tile_q0.  `next`: the slot whose lse comes next.
  auto vector_phase = [&](int tile_q0, int next) {
    if (ROLE == 0) {
      const float raw = NEAR ? 0.f : *raw_rows(next);   // asked for here, needed behind the exponentials
      const int q0_ = tile_q0 + row0;
      const bool some = tiles.some(q0_);
      if (some && !tiles.full(q0_)) {
#pragma unroll
        for (int half = 0; half < MB / 2; ++half)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) mask_rows32(s[2 * half][nb], s[2 * half + 1][nb], q0_ + 32 * half, g, qlo[nb], qhi[nb], true);
      }
      if (some) {
#pragma unroll
        for (int ch = 0; ch < MB / 2; ++ch)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            f32x4 &x = s[2 * ch][nb], &y = s[2 * ch + 1][nb];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              x[v] = __builtin_amdgcn_exp2f(x[v]);
              y[v] = __builtin_amdgcn_exp2f(y[v]);
            }
            ps[ch][nb] = pack_pair(x, y);
          }
      } else {   // for this pair alone there is nothing in the tile
#pragma unroll
        for (int ch = 0; ch < MB / 2; ++ch)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) ps[ch][nb] = zero_operand();
      }
      if (!NEAR) *raw_rows(next) = -lse_to_log2(raw);
#pragma unroll
      for (int ch = 0; ch < MB / 2; ++ch)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) hand[(ch * NB + nb) * 64] = ps[ch][nb];
      keep_order();
    } else {
      bf16x8 pr[MB / 2][NB];   // all of P first: one LDS round trip instead of one per operand
#pragma unroll
      for (int ch = 0; ch < MB / 2; ++ch)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) pr[ch][nb] = hand[(ch * NB + nb) * 64];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ch = 0; ch < MB / 2; ++ch)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          f32x4 &x = s[2 * ch][nb], &y = s[2 * ch + 1][nb];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            x[v] *= (float)pr[ch][nb][v];
            y[v] *= (float)pr[ch][nb][v + 4];
          }
          ps[ch][nb] = pack_pair(x, y);
        }
    }
  };
  // The barrier behind it: P has to be stored, while the AHEAD operands (two LDS reads each) fetched since stay in flight
  auto vector_barrier = [&]() {
    if (ROLE == 0 && NEAR) stores_loads_barrier<2 * AHEAD>();   // tile t+2
    else if (ROLE == 0) stores_barrier<2 * AHEAD>();
    else phase_barrier();
  };
  auto matrix_barrier = [&]() {
    if (!NEAR) wait_loads_barrier<LOADS>();      // tile t+2
    else if (ROLE == 1) wait_loads_barrier<0>();
    else phase_barrier();
  };

  if (walk.valid()) {   // uniform over the work-group: all waves take the same number of barriers
    const int ta = walk.cursor();
    issue(0);
    int tb = walk.cursor();
    issue(1);
    int tc = walk.cursor();
    if (!NEAR) issue(2);
    wait_loads_barrier<(NEAR ? 1 : 2) * LOADS>();   // tile 0
    if (ROLE == 1) phase_barrier();
    bf16x8 first[AHEAD];
    if (ROLE == 0) *raw_rows(0) = -lse_to_log2(*raw_rows(0));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) init_rows(0, mb);
    rows_fetch<D, MB, AHEAD>(rows_lds(0), ad, 0, first);
    rows_product<D, MB, NB, AHEAD>(rows_lds(0), ad, 0, xreg, s, init, first);
    wait_loads_barrier<NEAR ? 0 : LOADS>();       // tile 1
    if (NEAR && ROLE == 1) issue(2);
    vector_phase(ta, 1);
    cols_fetch<D, AHEAD>(cols_lds(0), ad, 0, first);
    vector_barrier();
    int slot = 0, tn = walk.cursor();
    uint32_t ql = q_lds(SLOTS - 1), ol = o_lds(SLOTS - 1), rl = lds0 + row_off(SLOTS - 1), ct = cols_lds(0), rt = rows_lds(1);
    if (!NEAR || ROLE == 0) walk.begin(wave, lane);
    float raw = 0.f;
    for (;;) {   // iteration t: tb, tc, tn are the first rows of tiles t+1, t+2, t+3
      // ---- matrix phase; everything else that an iteration computes stands behind its MFMAs or in the vector phase
      bf16x8 first_rows[AHEAD];
      constexpr int NCOLS = MB / 2 * DB;
      static_assert(LOADS <= NCOLS && MB <= NCOLS && AHEAD <= NCOLS, "a hook per operand");
      cols_product<D, MB / 2, NB, AHEAD>(ct, ad, 0, ps, acc, first, [&](int i) {
        if (i < LOADS && (!NEAR || ROLE == 0)) walk.load(i, ql, ol, rl, wave);
        if (NEAR && ROLE == 0 && i == 0) raw = *raw_rows(after(slot));
        if (NEAR && ROLE == 0 && i == NCOLS / 2 - 1) *raw_rows(after(slot)) = -lse_to_log2(raw);
        if (!BLK && (!NEAR || ROLE == 0)) {
#pragma unroll
          for (int part = 0; part < walk.PARTS; ++part)
            if (i == min(LOADS + part, NCOLS - 1)) walk.end(part);
        }
        if (i >= NCOLS - MB) init_rows(after(slot), i - (NCOLS - MB));
        if (i >= NCOLS - AHEAD) {
          const int f = i - (NCOLS - AHEAD);
          first_rows[f] = rows_operand<D>(rt, ad, 16 * (f % MB), f / MB);
        }
      });
      if (tb < 0) break;
      rows_product<D, MB, NB, AHEAD>(rt, ad, 0, xreg, s, init, first_rows);
      matrix_barrier();
      // ---- vector phase
      if (BLK && (!NEAR || ROLE == 0)) walk.advance();
      ql = q_lds(slot);
      ol = o_lds(slot);
      rl = lds0 + row_off(slot);
      const int left_slot = slot;
      slot = after(slot);
      ct = cols_lds(slot);
      rt = rows_lds(after(slot));
      const int tile_q0 = tb;
      tb = tc;
      tc = tn;
      tn = walk.cursor();
      if (NEAR) tc = tn;
      if (NEAR && ROLE == 1) issue(left_slot);
      else walk.begin(wave, lane);
      pin(slot, ql, ol, rl, ct, rt, tb, tc, tn);
      vector_phase(tile_q0, after(slot));
      cols_fetch<D, AHEAD>(ct, ad, 0, first);
      vector_barrier();
    }
    wait_global_loads();   // tiles past the end of the walk
    if (ROLE == 0) phase_barrier();
  }

  if (QS == 2) {   // the sums of pairs 2 and 3 through the tiles' LDS, which all waves have left
    static_assert(4 * DB * NB * 64 * 16 <= L::ROW_OFF, "the sums of four waves fit where the tiles were");
    f32x4* const sums = reinterpret_cast<f32x4*>(smem) + (2 * ROLE + (pair & 1)) * (DB * NB * 64) + lane;
    __syncthreads();
    if (pair >= 2) {
#pragma unroll
      for (int i = 0; i < DB * NB; ++i) sums[i * 64] = acc[i / NB][i % NB];
    }
    __syncthreads();
    if (pair >= 2) return;
#pragma unroll
    for (int i = 0; i < DB * NB; ++i) acc[i / NB][i % NB] += sums[i * 64];
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = k_w0 + 16 * nb + r;
    if (row >= sk) continue;
    const TensorDev& dst = ROLE == 0 ? st.dv : st.dk;
    const float mul = ROLE == 0 ? 1.f : -p.scale;   // (dS carried the other sign)
    float* out = (float*)dst.ptr + b * dst.sb + (int64_t)row * dst.ss + hk * dst.sh + 4 * g;
    f32x4 old[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) old[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (ROLE == 0 ? p.acc_dv : p.acc_dk) {   // all loads before the first store
#pragma unroll
      for (int db = 0; db < DB; ++db) old[db] = *reinterpret_cast<const f32x4*>(out + 16 * db);
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(out + 16 * db) = acc[db][nb] * mul + old[db];
  }
}

template <int D, bool BLK, bool MULTI, int BKV, bool TURNS>
__device__ __forceinline__ void dkdv_block(const BwdParams& p, char* smem, int block) {   // smem: laid out by DkdvLds, then the open flags
  int step = 0;   // the steps' work-groups one after the other
  while (MULTI && step + 1 < p.n_steps && block >= p.step[step + 1].first_block) ++step;
  const BwdStep& st = p.step[MULTI ? step : 0];
  const BlockMap bm = map_block<false>(block - st.first_block, p.batch * p.kv_heads, 1, st.k_runs.total(), st.k_side_by_side);
  if (!bm.valid) return;
  const int b = __builtin_amdgcn_readfirstlane(bm.key / p.kv_heads), hk = bm.key - b * p.kv_heads;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave < 4) dkdv_role<D, 0, BLK, BKV, TURNS>(p, st, smem, b, hk, bm.tile, wave);
  else dkdv_role<D, 1, BLK, BKV, TURNS>(p, st, smem, b, hk, bm.tile, wave);
}

// ---------------------------------------------------------------------------------------------
// Launches of few tiles (split_walks below): a work-group of four waves has 32 rows of dQ, or 32 key rows of dK and dV, and its
// waves deal the tiles of the other axis among themselves, each with two tiles in an LDS slot pair of its own and no barrier until the sums meet.
// What bounds such a launch is the chain of a walk (load, products, vector work, products), not a unit of the chip: it is four times
// shorter so, on eight (dQ) and two or four (dK/dV) times as many CUs.  A wave has up to 512 registers: K, V and both sums fit one.
template <int D>
struct SplitWalk {
  static constexpr int NW = 4, ROWS = 32, NB = ROWS / 16, DK = D / 32, DB = D / 16, AHEAD = 3;
  static constexpr int BT = 4096 / D, MB = BT / 16, TILE = BT * 2 * D;    // rows of a tile of the walked axis: 8 KiB of each tensor
  static constexpr int SLOT = 2 * TILE, WAVE = 2 * SLOT, VEC = BT * 4;
  static constexpr int VEC_OFF = NW * WAVE;                               // [wave][slot][lse, D]: 64 values, BT of them read
  static constexpr int BYTES = VEC_OFF + NW * 2 * 2 * 256;
  static constexpr int DBO = DB / NW;                                     // column blocks of a wave when the sums have met
};

// acc of the waves, at `sums` [wave][DB * NB][lane]: the sum of all for column blocks wave * DBO .. of this wave
template <int D>
__device__ __forceinline__ f32x4 split_sum(const f32x4* sums, int stride, int wave, int i, int nb) {
  using W = SplitWalk<D>;
  f32x4 x = sums[((wave * W::DBO + i) * W::NB + nb) * 64];
#pragma unroll
  for (int w = 1; w < W::NW; ++w) x += sums[w * stride + ((wave * W::DBO + i) * W::NB + nb) * 64];
  return x;
}
// Rows of a result from the waves' sums
template <int D>
__device__ __forceinline__ void split_store(const TensorDev& t, int b, int head, int row0, int rows, const f32x4* sums, int stride, float mul, int accumulate,
                                            int wave, int lane) {
  using W = SplitWalk<D>;
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int nb = 0; nb < W::NB; ++nb) {
    const int row = row0 + 16 * nb + r;
    if (row >= rows) continue;
    float* dst = (float*)t.ptr + b * t.sb + (int64_t)row * t.ss + head * t.sh + 16 * W::DBO * wave + 4 * g;
    f32x4 old[W::DBO];
#pragma unroll
    for (int i = 0; i < W::DBO; ++i) old[i] = accumulate ? *reinterpret_cast<const f32x4*>(dst + 16 * i) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < W::DBO; ++i) *reinterpret_cast<f32x4*>(dst + 16 * i) = split_sum<D>(sums + lane, stride, wave, i, nb) * mul + old[i];
  }
}

template <int D, bool MULTI>
__device__ __forceinline__ void dq_split_block(const BwdParams& p, char* smem, int block) {
  using W = SplitWalk<D>;
  constexpr int NB = W::NB, DK = W::DK, DB = W::DB, MB = W::MB, BT = W::BT, AHEAD = W::AHEAD;
  const int group = p.q_heads / p.kv_heads;
  const BlockMap bm = map_block<true>(block, p.batch * p.kv_heads, group, p.q_runs.total(), p.q_side_by_side);
  if (!bm.valid) return;
  const int b = __builtin_amdgcn_readfirstlane(bm.key / p.kv_heads), hk = bm.key - b * p.kv_heads, hq = hk * group + bm.head_in_group;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sq = p.sq, n_steps = MULTI ? p.n_steps : 1;
  const MaskDev q_side = p.step[0].mask;   // all steps have the same
  const int row0 = p.q_runs.tile_of(bm.tile) * W::ROWS, row1 = min(row0 + W::ROWS, sq);
  bf16x8 qreg[DK][NB], doreg[DK][NB];
  int q_pos[NB], klo[NB], khi[NB];
  float lse2[NB], dval[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = min(row0 + 16 * nb + r, sq - 1);
    q_pos[nb] = axis_position(axis_of<true>(q_side), row);
    const __bf16* qs = (const __bf16*)p.q.ptr + b * p.q.sb + hq * p.q.sh + (int64_t)row * p.q.ss + 8 * g;
    const __bf16* gs = (const __bf16*)p.d_o.ptr + b * p.d_o.sb + hq * p.d_o.sh + (int64_t)row * p.d_o.ss + 8 * g;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      qreg[ks][nb] = *reinterpret_cast<const bf16x8*>(qs + ks * 32);
      doreg[ks][nb] = *reinterpret_cast<const bf16x8*>(gs + ks * 32);
    }
    lse2[nb] = lse_to_log2(p.lse.ptr[b * p.lse.sb + hq * p.lse.sh + row]);
    dval[nb] = p.d.ptr[b * p.d.sb + hq * p.d.sh + row];
  }
  const float c = p.scale * kLog2e;
  f32x4 dq[DB][NB];
#pragma unroll
  for (int i = 0; i < DB * NB; ++i) dq[i / NB][i % NB] = f32x4{0.f, 0.f, 0.f, 0.f};
  int qlo, qhi;
  range_minmax<true>(q_side, row0, row1, qlo, qhi);
  OperandAddr<D> ad;
  ad.init(lane);
  const uint32_t lds = (uint32_t)(uintptr_t)(lds_bytes)smem + wave * W::WAVE;
  using Walk = KvStream<D, BT, 1, false, false>;
#pragma clang loop unroll(disable)
  for (int step = 0; step < n_steps; ++step) {
    const BwdStep& st = p.step[MULTI ? step : 0];
    const MaskDev mk = st.mask;
    const int sk = st.sk;
    const bool windowed = mk.window != kNoWindow;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) visible_rows<true>(mk, q_pos[nb], sk, klo[nb], khi[nb]);
    TileRanges tiles;
    tiles.init(row_intervals<false>(mk, qlo, qhi, sk, false), sk, BT);
    Walk walk;
    walk.init(mk, st.k, st.v, b, hk, sk, qlo, qhi, 0, lane, nullptr);
    wait_global_loads();
    walk.skip(wave);
    if (!walk.valid()) continue;
    auto ask = [&](uint32_t slot) {
      walk.begin(0, lane);
#pragma unroll
      for (int i = 0; i < Walk::N; ++i) walk.load_k(i, slot, 0);
#pragma unroll
      for (int i = 0; i < Walk::N; ++i) walk.load_v(i, slot + W::TILE, 0);
    };
    uint32_t slot = lds, other = lds + W::SLOT;
    ask(slot);
    for (;;) {
      const int k0 = walk.k0;
      walk.skip(W::NW);
      const bool more = walk.valid();
      if (more) {
        ask(other);
        wait_loads<Walk::LOADS>();
      } else {
        wait_loads<0>();
      }
      if (tiles.some(k0)) {
        f32x4 s[MB][NB], dp[MB][NB];
        bf16x8 ds[MB / 2][NB], first[AHEAD];
        rows_fetch<D, MB, AHEAD>(slot, ad, 0, first);
        rows_product_pair<D, MB, NB, AHEAD>(slot, slot + W::TILE, ad, qreg, doreg, s, dp, first);
        cols_fetch<D, AHEAD>(slot, ad, 0, first);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int ch = 0; ch < MB / 2; ++ch) {
            f32x4 &x = s[2 * ch][nb], &y = s[2 * ch + 1][nb];
            if (!tiles.full(k0)) mask_rows32(x, y, k0 + 32 * ch, g, klo[nb], khi[nb], windowed);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              x[v] = __builtin_amdgcn_exp2f(c * x[v] - lse2[nb]) * (dp[2 * ch][nb][v] - dval[nb]);
              y[v] = __builtin_amdgcn_exp2f(c * y[v] - lse2[nb]) * (dp[2 * ch + 1][nb][v] - dval[nb]);
            }
            ds[ch][nb] = pack_pair(x, y);
          }
        cols_product<D, MB / 2, NB, AHEAD>(slot, ad, 0, ds, dq, first);
      }
      if (!more) break;
      const uint32_t x = slot;
      slot = other;
      other = x;
    }
  }
  f32x4* const sums = reinterpret_cast<f32x4*>(smem);
  constexpr int STRIDE = W::WAVE / 16;
  static_assert(DB * NB * 64 <= STRIDE, "a wave's sums fit where its tiles were");
#pragma unroll
  for (int i = 0; i < DB * NB; ++i) sums[wave * STRIDE + i * 64 + lane] = dq[i / NB][i % NB];
  __syncthreads();
  split_store<D>(p.dq, b, hq, row0, sq, sums, STRIDE, p.scale, p.acc_dq, wave, lane);
}

template <int D, bool MULTI>
__device__ __forceinline__ void dkdv_split_block(const BwdParams& p, char* smem, int block) {
  using W = SplitWalk<D>;
  constexpr int NB = W::NB, DK = W::DK, DB = W::DB, MB = W::MB, BT = W::BT, AHEAD = W::AHEAD;
  int step = 0;   // the steps' work-groups one after the other
  while (MULTI && step + 1 < p.n_steps && block >= p.step[step + 1].first_block) ++step;
  const BwdStep& st = p.step[MULTI ? step : 0];
  const BlockMap bm = map_block<false>(block - st.first_block, p.batch * p.kv_heads, 1, st.k_runs.total(), st.k_side_by_side);
  if (!bm.valid) return;
  const int b = __builtin_amdgcn_readfirstlane(bm.key / p.kv_heads), hk = bm.key - b * p.kv_heads, group = p.q_heads / p.kv_heads;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sq = p.sq, sk = st.sk;
  const MaskDev mk = st.mask;
  const int row0 = st.k_runs.tile_of(bm.tile) * W::ROWS, row1 = min(row0 + W::ROWS, sk);
  const float c = p.scale * kLog2e;
  // scale * log2(e) * K and -V, as in dkdv_role
  bf16x8 kreg[DK][NB], vreg[DK][NB];
  int qlo[NB], qhi[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int row = min(row0 + 16 * nb + r, sk - 1);
    visible_rows<false>(mk, axis_position(axis_of<false>(mk), row), sq, qlo[nb], qhi[nb]);
    const __bf16* ks_ = (const __bf16*)st.k.ptr + b * st.k.sb + hk * st.k.sh + (int64_t)row * st.k.ss + 8 * g;
    const __bf16* vs_ = (const __bf16*)st.v.ptr + b * st.v.sb + hk * st.v.sh + (int64_t)row * st.v.ss + 8 * g;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      kreg[ks][nb] = *reinterpret_cast<const bf16x8*>(ks_ + ks * 32);
      vreg[ks][nb] = *reinterpret_cast<const bf16x8*>(vs_ + ks * 32);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        kreg[ks][nb][e] = (__bf16)((float)kreg[ks][nb][e] * c);
        vreg[ks][nb][e] = -vreg[ks][nb][e];
      }
    }
  }
  f32x4 dk[DB][NB], dv[DB][NB];
#pragma unroll
  for (int i = 0; i < DB * NB; ++i) dk[i / NB][i % NB] = dv[i / NB][i % NB] = f32x4{0.f, 0.f, 0.f, 0.f};
  int lo, hi;
  range_minmax<false>(mk, row0, row1, lo, hi);
  TileRanges tiles;
  tiles.init(row_intervals<true>(mk, lo, hi, sq, false), sq, BT);
  const TileRun run = visible_tiles<true, BT>(mk, lo, hi, sq);
  const int start = __builtin_amdgcn_readfirstlane(run.start), len = __builtin_amdgcn_readfirstlane(run.len);
  OperandAddr<D> ad;
  ad.init(lane);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_bytes)smem, lds = lds0 + wave * W::WAVE;
  const uint32_t vec_off = W::VEC_OFF + wave * 2 * 512;
  // The walk: head after head, the tiles wave, wave + NW, .. of each (heads take turns in which wave starts)
  using Stager = DirectStager<D, BT, 1>;
  constexpr int LOADS = 2 * Stager::N + 2;
  Stager q_rows, o_rows;
  uint32_t vec_lane = 0;
  const char *q_head = reinterpret_cast<const char*>((const __bf16*)p.q.ptr + b * p.q.sb + hk * group * p.q.sh);
  const char *o_head = reinterpret_cast<const char*>((const __bf16*)p.d_o.ptr + b * p.d_o.sb + hk * group * p.d_o.sh);
  const char *l_head = reinterpret_cast<const char*>(p.lse.ptr + b * p.lse.sb + hk * group * p.lse.sh);
  const char *d_head = reinterpret_cast<const char*>(p.d.ptr + b * p.d.sb + hk * group * p.d.sh);
  int valid = 0;   // rows the lanes' offsets are clamped to
  int head = 0, at = wave;
  auto settle = [&]() {   // to the next tile there is; head == group: none
    while (head < group && at >= len) {
      at -= len;
      ++head;
    }
    pin(head, at);
  };
  auto ask = [&](int n) {   // the cursor's tile into slot n
    const int first_row = (start + at) * BT, rows = min(sq - first_row, BT);
    if (rows != valid) {
      valid = rows;
      q_rows.clamp(p.q.ss, rows, 0, lane);
      o_rows.clamp(p.d_o.ss, rows, 0, lane);
      vec_lane = 4u * (uint32_t)min(lane, rows - 1);
    }
    const char* q_tile = q_head + 2 * ((int64_t)head * p.q.sh + (int64_t)first_row * p.q.ss);
    const char* o_tile = o_head + 2 * ((int64_t)head * p.d_o.sh + (int64_t)first_row * p.d_o.ss);
    const char* l_tile = l_head + 4 * ((int64_t)head * p.lse.sh + first_row);
    const char* d_tile = d_head + 4 * ((int64_t)head * p.d.sh + first_row);
    pin(q_tile, o_tile, l_tile, d_tile);
    const uint32_t q_lds = lds + n * W::SLOT, vec = lds0 + vec_off + n * 512;
    load_dword_to_lds(l_tile, vec_lane, vec);
    load_dword_to_lds(d_tile, vec_lane, vec + 256);
#pragma unroll
    for (int i = 0; i < Stager::N; ++i) q_rows.load_one(q_tile, i, q_lds, 0);
#pragma unroll
    for (int i = 0; i < Stager::N; ++i) o_rows.load_one(o_tile, i, q_lds + W::TILE, 0);
  };
  wait_global_loads();
  if (len > 0) settle();
  else head = group;
  if (head < group) {
    int n = 0;
    ask(0);
    for (;;) {
      const int q0 = (start + at) * BT;
      at += W::NW;
      settle();
      const bool more = head < group;
      if (more) {
        ask(n ^ 1);
        wait_loads<LOADS>();
      } else {
        wait_loads<0>();
      }
      if (tiles.some(q0)) {
        const uint32_t qt = lds + n * W::SLOT, ot = qt + W::TILE;
        const char* vec = smem + vec_off + n * 512;
        f32x4 s[MB][NB], dp[MB][NB], init[MB];
        bf16x8 pp[MB / 2][NB], ds[MB / 2][NB], first[AHEAD];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(vec + 4 * (16 * mb + 4 * g));
#pragma unroll
          for (int v = 0; v < 4; ++v) init[mb][v] = -lse_to_log2(x[v]);
        }
        rows_fetch<D, MB, AHEAD>(qt, ad, 0, first);
        rows_product<D, MB, NB, AHEAD>(qt, ad, 0, kreg, s, init, first);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) init[mb] = *reinterpret_cast<const f32x4*>(vec + 256 + 4 * (16 * mb + 4 * g));
        rows_fetch<D, MB, AHEAD>(ot, ad, 0, first);
        rows_product<D, MB, NB, AHEAD>(ot, ad, 0, vreg, dp, init, first);   // D - dP
        cols_fetch<D, AHEAD>(ot, ad, 0, first);
#pragma unroll
        for (int ch = 0; ch < MB / 2; ++ch)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            f32x4 &x = s[2 * ch][nb], &y = s[2 * ch + 1][nb], &dx = dp[2 * ch][nb], &dy = dp[2 * ch + 1][nb];
            if (!tiles.full(q0)) mask_rows32(x, y, q0 + 32 * ch, g, qlo[nb], qhi[nb], true);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              x[v] = __builtin_amdgcn_exp2f(x[v]);
              y[v] = __builtin_amdgcn_exp2f(y[v]);
            }
            pp[ch][nb] = pack_pair(x, y);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              dx[v] *= (float)pp[ch][nb][v];
              dy[v] *= (float)pp[ch][nb][v + 4];
            }
            ds[ch][nb] = pack_pair(dx, dy);   // -dS
          }
        cols_product<D, MB / 2, NB, AHEAD>(ot, ad, 0, pp, dv, first);
        cols_fetch<D, AHEAD>(qt, ad, 0, first);
        cols_product<D, MB / 2, NB, AHEAD>(qt, ad, 0, ds, dk, first);
      }
      if (!more) break;
      n ^= 1;
    }
  }
  f32x4* const sums = reinterpret_cast<f32x4*>(smem);
  constexpr int STRIDE = W::WAVE / 16, HALF = DB * NB * 64;
  static_assert(2 * HALF <= STRIDE, "a wave's sums fit where its tiles were");
#pragma unroll
  for (int i = 0; i < DB * NB; ++i) {
    sums[wave * STRIDE + i * 64 + lane] = dk[i / NB][i % NB];
    sums[wave * STRIDE + HALF + i * 64 + lane] = dv[i / NB][i % NB];
  }
  __syncthreads();
  split_store<D>(st.dk, b, hk, row0, sk, sums, STRIDE, -p.scale, p.acc_dk, wave, lane);
  split_store<D>(st.dv, b, hk, row0, sk, sums + HALF, STRIDE, 1.f, p.acc_dv, wave, lane);
}

// ---------------------------------------------------------------------------------------------
// A kernel argument indexed with a variable would be copied to scratch memory: several steps are read through the argument
// pointer, a single one (MULTI false) directly, all at once at the start.
__device__ __forceinline__ const BwdParams& launch_args() {
  typedef const __attribute__((address_space(4))) BwdParams* args_ptr;
  return *(const BwdParams*)(args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
}
template <int D, int NW, bool BLK, bool MULTI>
__global__ __launch_bounds__(64 * NW, D == 128 ? 1 : 3) void step_bwd_dq_kernel(BwdParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int AHEAD = BLK ? 3 : kAhead16;   // (the block flags take the registers of one operand)
  if constexpr (MULTI) dq_block<D, NW, BLK, true, AHEAD, D == 128>(launch_args(), smem, blockIdx.x);
  else dq_block<D, NW, BLK, false, AHEAD, D == 128>(p, smem, blockIdx.x);
}
template <int D, bool BLK, bool MULTI, int BKV, bool TURNS>
__global__ __launch_bounds__(512, TURNS ? 1 : 4) void step_bwd_dkdv_kernel(BwdParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if constexpr (MULTI) dkdv_block<D, BLK, true, BKV, TURNS>(launch_args(), smem, blockIdx.x);
  else dkdv_block<D, BLK, false, BKV, TURNS>(p, smem, blockIdx.x);
}
// Both in one launch (they share nothing but inputs): the first n_first work-groups (a multiple of 8, as the mapping to
// XCDs needs) are those of the kernel whose walks are the longer ones.
template <int D, bool MULTI, int BKV, bool TURNS>
__global__ __launch_bounds__(512, TURNS ? 1 : 4) void step_bwd_both_kernel(BwdParams, int n_first, int dq_first) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // each side reads its own arguments: loaded for both at the start they would not fit the scalar registers
  typedef const __attribute__((address_space(4))) BwdParams* args_ptr;
  args_ptr args = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  const int in_first = (int)blockIdx.x < n_first, block = blockIdx.x - (in_first ? 0 : n_first);
  if (in_first != dq_first) {
    asm volatile("" : "+s"(args));
    dkdv_block<D, false, MULTI, BKV, TURNS>(*(const BwdParams*)args, smem, block);
  } else {
    asm volatile("" : "+s"(args));
    dq_block<D, 8, false, MULTI, TURNS ? 3 : 2, TURNS>(*(const BwdParams*)args, smem, block);
  }
}

// Both with walks dealt to the waves of a work-group
template <int D, bool MULTI>
__global__ __launch_bounds__(64 * SplitWalk<D>::NW, 1) void step_bwd_split_kernel(BwdParams, int n_first, int dq_first) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  typedef const __attribute__((address_space(4))) BwdParams* args_ptr;
  args_ptr args = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  const int in_first = (int)blockIdx.x < n_first, block = blockIdx.x - (in_first ? 0 : n_first);
  if (in_first != dq_first) {
    asm volatile("" : "+s"(args));
    dkdv_split_block<D, MULTI>(*(const BwdParams*)args, smem, block);
  } else {
    asm volatile("" : "+s"(args));
    dq_split_block<D, MULTI>(*(const BwdParams*)args, smem, block);
  }
}

// Whether the dK/dV kernel takes key tiles of 64 rows.  A tile of 64 costs 0.6-0.7 of one of 128 (more barriers and LDS
// traffic per MFMA), so it pays where the tiles of 128 leave half the CUs idle, and, up to one per CU, where the walks
// are uneven, as the mask makes them, and the longest one decides.  One step, full mask, tiles of 128: 64 of them 61 us
// against 45 with tiles of 64, 128 (16/2 heads, 8192 rows) 1556 against 1125, but 160 258 against 332, 256 68 against
// 82.  Own shard, causal: 160 252 against 169, 256 63 against 53, 288 87 against 81, 384 48 against 54.
static bool narrow_key_tiles(const BwdParams& p) {
  int n = 0;
  bool uneven = false;
  for (int i = 0; i < p.n_steps; ++i) {
    const BwdStep& st = p.step[i];
    n += p.batch * p.kv_heads * st.k_runs.total();
    uneven |= uneven_k_walks(st.mask, p.sq, st.sk, st.k_runs, 128);
  }
  if (p.step[0].mask.blk || n == 0 || n > 256) return false;
  return n <= 128 || uneven;
}

// The work-groups of a kernel: the tiles that see something, and zeros into what gets no work-group under "=".
static hipError_t plan_dq(BwdParams& p, int BQ, hipStream_t stream, LaunchLog* log) {
  p.q_runs = nonempty_q_runs(p.step, p.n_steps, p.sq, BQ);
  p.q_side_by_side = q_side_by_side(p.step, p.n_steps, p.sq, p.batch * p.kv_heads, p.q_heads / p.kv_heads, p.q_runs, BQ);
  if (!log && !p.acc_dq && p.q_runs.total() < (p.sq + BQ - 1) / BQ)
    return launch_zero_tensor(p.dq, p.batch, p.sq, p.q_heads, p.head_dim, stream);
  return hipSuccess;
}
static hipError_t plan_dkdv_tiles(BwdParams& p, int tile, hipStream_t stream, LaunchLog* log) {
  const int n_keys = p.batch * p.kv_heads;
  for (int i = 0; i < p.n_steps; ++i) {
    BwdStep& st = p.step[i];
    st.k_runs = nonempty_k_runs(st.mask, p.sq, st.sk, tile);
    st.k_side_by_side = k_side_by_side(st.mask, p.sq, st.sk, n_keys, st.k_runs, tile);
    if (!log && st.k_runs.total() < (st.sk + tile - 1) / tile) {
      hipError_t e = hipSuccess;
      if (!p.acc_dk) e = launch_zero_tensor(st.dk, p.batch, st.sk, p.kv_heads, p.head_dim, stream);
      if (e == hipSuccess && !p.acc_dv) e = launch_zero_tensor(st.dv, p.batch, st.sk, p.kv_heads, p.head_dim, stream);
      if (e != hipSuccess) return e;
    }
  }
  // heaviest first among the steps, too
  if (p.n_steps > 1) {
    auto longest = [&](const BwdStep& st) {
      return st.k_runs.total() ? k_tile_walk(st.mask, p.sq, st.sk, st.k_runs.tile_of(0), tile) : 0;
    };
    std::stable_sort(p.step, p.step + p.n_steps, [&](const BwdStep& x, const BwdStep& y) { return longest(x) > longest(y); });
  }
  int block = 0;
  for (int i = 0; i < p.n_steps; ++i) {
    p.step[i].first_block = block;
    block += mapped_grid(n_keys, 1, p.step[i].k_runs.total());
  }
  return hipSuccess;
}
static hipError_t plan_dkdv(BwdParams& p, bool& narrow, hipStream_t stream, LaunchLog* log) {
  for (int i = 0; i < p.n_steps; ++i) p.step[i].k_runs = nonempty_k_runs(p.step[i].mask, p.sq, p.step[i].sk, 128);
  narrow = narrow_key_tiles(p);
  return plan_dkdv_tiles(p, narrow ? 64 : 128, stream, log);
}
static int dq_grid(const BwdParams& p) { return mapped_grid(p.batch * p.kv_heads, p.q_heads / p.kv_heads, p.q_runs.total()); }
static int dkdv_grid(const BwdParams& p) {
  const BwdStep& last = p.step[p.n_steps - 1];
  return last.first_block + mapped_grid(p.batch * p.kv_heads, 1, last.k_runs.total());
}

// a dQ work-group walks every step (three products a tile against two), a dK/dV one the heads of its group
static bool longer_dq_walks(const BwdParams& p) { return p.n_steps > 1 && 3 * p.n_steps > 4 * (p.q_heads / p.kv_heads); }

template <int D>
constexpr int kDqLds = kBwdSlots<D == 128> * 2 * 64 * 2 * D;
template <int D, bool TURNS>
constexpr int kDkdvLds = DkdvLds<D, TURNS>::BYTES;
constexpr int kFlagsLds = kMaxBlockCacheTiles;   // with a block mask
constexpr int kAlone = 256;   // work-groups that have a CU for themselves

template <int D>
static hipError_t launch_dq_t(BwdParams& p, hipStream_t stream, LaunchLog* log) {
  const hipError_t e = plan_dq(p, 32 * kDqWaves<D>, stream, log);
  const int grid = dq_grid(p);
  if (e != hipSuccess || grid == 0) return e;
  if (log) {
    log->push_back(BURST_KERNEL_DQ);
    return hipSuccess;
  }
  constexpr int NW = kDqWaves<D>, NT = 64 * NW;
  if (p.step[0].mask.blk) hipLaunchKernelGGL((step_bwd_dq_kernel<D, NW, true, false>), dim3(grid), dim3(NT), kDqLds<D> + kFlagsLds, stream, p);
  else if (p.n_steps > 1) hipLaunchKernelGGL((step_bwd_dq_kernel<D, NW, false, true>), dim3(grid), dim3(NT), kDqLds<D>, stream, p);
  else hipLaunchKernelGGL((step_bwd_dq_kernel<D, NW, false, false>), dim3(grid), dim3(NT), kDqLds<D>, stream, p);
  return hipGetLastError();
}

template <int D, bool BLK, bool MULTI, int BKV, bool TURNS>
static void launch_dkdv_kernel(const BwdParams& p, int grid, hipStream_t stream) {
  constexpr int LDS = kDkdvLds<D, TURNS> + (BLK ? kFlagsLds : 0);
  static_assert((TURNS ? 1 : 2) * LDS <= 160 * 1024, "LDS of a CU");
  hipLaunchKernelGGL((step_bwd_dkdv_kernel<D, BLK, MULTI, BKV, TURNS>), dim3(grid), dim3(512), LDS, stream, p);
}
template <int D>
static hipError_t launch_dkdv_t(BwdParams& p, hipStream_t stream, LaunchLog* log) {
  bool narrow = false;
  const hipError_t e = plan_dkdv(p, narrow, stream, log);
  const int grid = dkdv_grid(p);
  if (e != hipSuccess || grid == 0) return e;
  const bool multi = p.n_steps > 1, alone = D == 128 || p.step[0].mask.blk || narrow || grid <= kAlone;
  if (log) {
    log->push_back(BURST_KERNEL_DKDV | (narrow ? BURST_KERNEL_KEY_TILES_64 : 0) | (alone ? 0 : BURST_KERNEL_SHARED_CU));
    return hipSuccess;
  }
  if (p.step[0].mask.blk) launch_dkdv_kernel<D, true, false, 128, true>(p, grid, stream);
  else if (narrow && multi) launch_dkdv_kernel<D, false, true, 64, true>(p, grid, stream);
  else if (narrow) launch_dkdv_kernel<D, false, false, 64, true>(p, grid, stream);
  else if (alone) multi ? launch_dkdv_kernel<D, false, true, 128, true>(p, grid, stream)
                        : launch_dkdv_kernel<D, false, false, 128, true>(p, grid, stream);
  else if constexpr (D == 64) multi ? launch_dkdv_kernel<D, false, true, 128, false>(p, grid, stream)
                                    : launch_dkdv_kernel<D, false, false, 128, false>(p, grid, stream);
  return hipGetLastError();
}

// Work-groups (dQ tiles of 256 rows and key tiles of 128) up to which a step's two kernels go out as one launch: the
// second one's work-groups then fill the CUs that the last round of the first leaves idle, and there is one start
// less.  One step, d = 128, two launches against one: 6 work-groups 33 -> 21 us, 4 heads x 2048 rows (96) 115 -> 78,
// 12 heads x 3000 (432) 262 -> 189, 48 x 1500 (864) 260 -> 217, causal 16 x 6000 (1136) 479 -> 446; alike from 32 x 4096
// (1536) on, 772 and 770, causal 422 and 428.  Several steps, twice as many: they go from longer to shorter walks, which a
// part-empty round costs more.  Apart, dK/dV's first, dQ's first: 3 steps of 48 x 1500 rows, d = 64 (2016) 365, 334, 295 us;
// 8 of 16/2 heads x 8192 (1344), whose key tiles walk 8 heads, 5861, 5771, 5947; 4 of 32 x 4096 (3584) 1591, 1583, 1636.
constexpr int kBothLaunch = 1280, kBothBQ = 256;   // (query rows of its dQ work-groups)

// Whether the work-groups of a joint launch at d = 64 share CUs (two of up to 128 registers) instead of having one each: a shared CU
// does more in a time, and each of its work-groups less.  So it pays where there are several times as many as CUs, and not where the
// longest walks decide: the work of all has to be 1.1 times that of a longest one on every CU, and twice where the walks are uneven
// (they are launched longest first, and sharing holds up just those).  In units of a product of 64 x 128 rows; first and last tile
// stand for all.  us with a CU each and shared, by that measure: even 2.6 (4 x 12 heads x 1500 rows, full) 134, 118; 1.8 (8 x 12 x
// 512) 49, 41; 1.2 (2 x 16 x 1000, two steps) 75, 68; uneven 4.6 (4 x 64/32 x 576, two steps) 164, 124; 2.2 (4 x 12 x 1500, three
// steps) 294, 258; 1.7 (16 x 6000 causal) 267, 284; 0.4 (8 x 2048, zigzag, four steps) 148, 180.
static bool crowded(const BwdParams& p, bool narrow) {
  const int group = p.q_heads / p.kv_heads, tile = narrow ? 64 : 128, keys = p.batch * p.kv_heads;
  int64_t first = 0, last = 0, total = 0, longest = 0;
  bool uneven = uneven_q_walks(p.step, p.n_steps, p.sq, p.q_runs, kBothBQ);
  for (int i = 0, nq = p.q_runs.total(); i < p.n_steps && nq > 0; ++i) {
    first += 6 * q_tile_walk(p.step[i].mask, p.sq, p.step[i].sk, p.q_runs.tile_of(nq - 1), kBothBQ);
    last += 6 * q_tile_walk(p.step[i].mask, p.sq, p.step[i].sk, p.q_runs.tile_of(0), kBothBQ);
  }
  total = (int64_t)keys * group * p.q_runs.total() * (first + last) / 2;
  longest = first;
  for (int i = 0; i < p.n_steps; ++i) {
    const BwdStep& st = p.step[i];
    const int n = st.k_runs.total();
    if (n == 0) continue;
    const int64_t per = (narrow ? 2 : 4) * group;
    first = per * k_tile_walk(st.mask, p.sq, st.sk, st.k_runs.tile_of(0), tile);
    last = per * k_tile_walk(st.mask, p.sq, st.sk, st.k_runs.tile_of(n - 1), tile);
    total += (int64_t)keys * n * (first + last) / 2;
    longest = std::max(longest, first);
    uneven |= 2 * last <= first;
  }
  return 10 * total >= (uneven ? 20 : 11) * kAlone * longest;
}
template <int D, bool MULTI, int BKV, bool TURNS>
static void launch_both_kernel(const BwdParams& p, int grid, int n_first, int dq_first, hipStream_t stream) {
  constexpr int DQ_LDS = kBwdSlots<TURNS> * 2 * 64 * 2 * D, LDS = std::max(kDkdvLds<D, TURNS>, DQ_LDS);
  hipLaunchKernelGGL((step_bwd_both_kernel<D, MULTI, BKV, TURNS>), dim3(grid), dim3(512), LDS, stream, p, n_first, dq_first);
}
// Whether the walks of a joint launch are dealt to the waves of its work-groups.  By the time of the longest walk or, if longer,
// of the work spread over the CUs, in products of a wave (a product of 64 x 32; d = 128 0.3 us, d = 64 0.15): three for a tile of dQ, four for one
// of dK/dV, and about eight to start a further work-group on a CU.  The other kernels' work-groups have a CU each: a tile costs dQ, for 256
// rows, 6 (d = 64: 8) of them, and dK/dV, whose waves share a tile as it is, 3 (4).  So splitting pays by dQ's walks and for few of them.
// us of backward with D and fills, d = 128 (d = 64): full 2 x 256 rows 35.9, 27.9 (28.0, 23.5); 4 x 1024 59.0, 45.5 (43.6, 32.0); 1 x 4096 140, 98 (97.5,
// 56.7); 8 x 1024 62.7, 61.7 (44.7, 41.7); 12 x 1024 67.8, 89.3 (47.2, 55.8); 64 x 128 32.0, 37.1 (25.1, 29.8); 8/1 x 1024 132, 164 (91, 88); causal 8 x
// 1024 62.4, 53.0 (45.0, 38.3); 1 x 16384 512, 498 (344, 265); 1 x 24576 976, 1075 (631, 556); 12 x 1500 93.7, 106 (67.6, 73.4).
template <int D>
static bool split_walks(const BwdParams& p) {
  constexpr int ROWS = SplitWalk<D>::ROWS, kStart = 8, kDq = D == 128 ? 6 : 8, kDkdv = D == 128 ? 3 : 4;
  const int64_t keys = (int64_t)p.batch * p.kv_heads, group = p.q_heads / p.kv_heads;
  const Walks q = q_walks(p.step, p.n_steps, p.sq, ROWS);
  int64_t groups = keys * group * q.tiles, work = 3 * keys * group * q.total, dkdv = 0;
  for (int i = 0; i < p.n_steps; ++i) {
    const Walks k = k_walks(p.step[i].mask, p.sq, p.step[i].sk, ROWS);
    groups += keys * k.tiles;
    work += 4 * keys * group * k.total;
    dkdv = std::max(dkdv, group * k.longest);
  }
  if (q.longest == 0) return false;
  return std::max({3 * q.longest, 4 * dkdv, work / kAlone}) + (groups - 1) / kAlone * kStart <= std::max(kDq * q.longest, kDkdv * dkdv);
}
template <int D>
static hipError_t launch_split_t(BwdParams& p, hipStream_t stream, LaunchLog* log) {
  using W = SplitWalk<D>;
  hipError_t e = plan_dq(p, W::ROWS, stream, log);
  if (e == hipSuccess) e = plan_dkdv_tiles(p, W::ROWS, stream, log);
  const int n_dkdv = dkdv_grid(p), n_dq = dq_grid(p), grid = n_dkdv + n_dq;
  if (e != hipSuccess || grid == 0) return e;
  if (log) {
    log->push_back(BURST_KERNEL_DQ | BURST_KERNEL_DKDV | BURST_KERNEL_DEALT);
    return hipSuccess;
  }
  const int dq_first = longer_dq_walks(p), n_first = dq_first ? n_dq : n_dkdv;
  if (p.n_steps > 1) hipLaunchKernelGGL((step_bwd_split_kernel<D, true>), dim3(grid), dim3(64 * W::NW), W::BYTES, stream, p, n_first, dq_first);
  else hipLaunchKernelGGL((step_bwd_split_kernel<D, false>), dim3(grid), dim3(64 * W::NW), W::BYTES, stream, p, n_first, dq_first);
  return hipGetLastError();
}
// One launch of both kernels; `done` says whether it was taken.
template <int D>
static hipError_t launch_both_t(BwdParams& p, bool& done, hipStream_t stream, LaunchLog* log) {
  const int n_keys = p.batch * p.kv_heads, group = p.q_heads / p.kv_heads;
  int64_t most = (int64_t)n_keys * group * ((p.sq + kBothBQ - 1) / kBothBQ);
  for (int i = 0; i < p.n_steps; ++i) most += (int64_t)n_keys * ((p.step[i].sk + 127) / 128);
  done = most <= (p.n_steps > 1 ? 2 : 1) * kBothLaunch;
  if (!done) return hipSuccess;
  if (split_walks<D>(p)) return launch_split_t<D>(p, stream, log);
  bool narrow = false;
  hipError_t e = plan_dq(p, kBothBQ, stream, log);
  if (e == hipSuccess) e = plan_dkdv(p, narrow, stream, log);
  const int n_dkdv = dkdv_grid(p), n_dq = dq_grid(p), grid = n_dkdv + n_dq;
  if (e != hipSuccess || grid == 0) return e;
  const int dq_first = longer_dq_walks(p), n_first = dq_first ? n_dq : n_dkdv;
  const bool multi = p.n_steps > 1;
  const bool alone = D == 128 || grid <= kAlone || !crowded(p, narrow);
  if (log) {
    log->push_back(BURST_KERNEL_DQ | BURST_KERNEL_DKDV | (narrow ? BURST_KERNEL_KEY_TILES_64 : 0) | (alone ? 0 : BURST_KERNEL_SHARED_CU));
    return hipSuccess;
  }
  auto launch = [&](auto m, auto bkv) {
    if (alone) launch_both_kernel<D, m.value, bkv.value, true>(p, grid, n_first, dq_first, stream);
    else if constexpr (D == 64) launch_both_kernel<D, m.value, bkv.value, false>(p, grid, n_first, dq_first, stream);
  };
  using narrow_tile = std::integral_constant<int, 64>;
  using wide_tile = std::integral_constant<int, 128>;
  if (narrow && multi) launch(std::true_type(), narrow_tile());
  else if (narrow) launch(std::false_type(), narrow_tile());
  else if (multi) launch(std::true_type(), wide_tile());
  else launch(std::false_type(), wide_tile());
  return hipGetLastError();
}

template <int D>
static hipError_t launch_bwd_groups(const BwdParams& p0, const BwdStep* steps, int n, hipStream_t stream, LaunchLog* log) {
  BwdParams p = p0;
  const bool dkdv = steps[0].dk.ptr != nullptr;
  hipError_t e = hipSuccess;
  std::vector<BwdStep> whole;   // the steps of which some query row sees something
  for (int i = 0; i < n; ++i) {
    const BwdStep& st = steps[i];
    if (classify(st.mask, 0, p.sq, 0, st.sk, false) != TILE_SKIP) {
      whole.push_back(st);
      continue;
    }
    if (log) continue;
    if (dkdv && !p.acc_dk) e = launch_zero_tensor(st.dk, p.batch, st.sk, p.kv_heads, p.head_dim, stream);
    if (e == hipSuccess && dkdv && !p.acc_dv) e = launch_zero_tensor(st.dv, p.batch, st.sk, p.kv_heads, p.head_dim, stream);
    if (e != hipSuccess) return e;
  }
  n = (int)whole.size();
  if (n == 0) return !log && p.dq.ptr && !p.acc_dq ? launch_zero_tensor(p.dq, p.batch, p.sq, p.q_heads, p.head_dim, stream) : hipSuccess;
  bool together = p.dq.ptr && dkdv && p.sq <= chunk_rows();
  for (const BwdStep& st : whole) together = together && !st.mask.blk && st.sk <= chunk_rows();
  auto put = [&](const std::vector<BwdStep>& from, int first, int end) {
    p.n_steps = end - first;
    std::copy(from.begin() + first, from.begin() + end, p.step);
  };
  if (together && n <= kMaxSteps) {
    bool done = false;
    put(whole, 0, n);
    e = launch_both_t<D>(p, done, stream, log);
    if (done) return e;
  }
  if (p0.dq.ptr) {   // the dQ kernel streams the key axis
    std::vector<BwdStep> parts;
    for (const BwdStep& step : whole) {
      const MaskDev& mk = step.mask;
      const std::vector<RowRange> ranges = chunk_ranges(mk.k_nseg, mk.k_seg_len, step.sk, mk.blk ? mk.blk_k : 0);
      for (const RowRange& rg : ranges) {
        BwdStep st = step;
        if (ranges.size() > 1) {
          st.mask = sub_mask<false>(mk, rg.r0, rg.r1);
          st.sk = rg.r1 - rg.r0;
          offset_rows(st.k, rg.r0);
          offset_rows(st.v, rg.r0);
        }
        parts.push_back(st);
      }
    }
    bool any = false;
    e = for_step_groups(parts, p.sq, p.batch * p.q_heads, [&](int first, int end) {
      put(parts, first, end);
      const hipError_t err = launch_dq_t<D>(p, stream, log);
      p.acc_dq = 1;
      any = true;
      return err;
    });
    if (e == hipSuccess && !any && !p0.acc_dq && !log) e = launch_zero_tensor(p.dq, p.batch, p.sq, p.q_heads, p.head_dim, stream);
    if (e != hipSuccess) return e;
  }
  if (dkdv) {   // the dK/dV kernel streams the query axis
    const MaskDev mk = whole[0].mask;   // all steps have the same query side
    const std::vector<RowRange> ranges = chunk_ranges(mk.q_nseg, mk.q_seg_len, p0.sq, mk.blk ? mk.blk_q : 0);
    for (const RowRange& rg : ranges) {
      p = p0;
      std::vector<BwdStep> parts = whole;
      if (ranges.size() > 1) {
        for (BwdStep& st : parts) st.mask = sub_mask<true>(st.mask, rg.r0, rg.r1);
        p.sq = rg.r1 - rg.r0;
        offset_rows(p.q, rg.r0);
        offset_rows(p.d_o, rg.r0);
        p.lse.ptr += rg.r0;
        p.d.ptr += rg.r0;
        if (&rg != &ranges.front()) p.acc_dk = p.acc_dv = 1;
      }
      auto share = [&](const BwdStep& st) {
        return !st.mask.blk && (share_launch(p.batch * p.kv_heads, st.sk) ||
                                p.q_heads / p.kv_heads * longest_k_walk(st.mask, p.sq, st.sk) <= kShareKeyWalk);
      };
      for (int first = 0, end; first < n; first = end) {
        for (end = first + 1; end < n && end - first < kMaxSteps && share(parts[first]) && share(parts[end]);) ++end;
        put(parts, first, end);
        e = launch_dkdv_t<D>(p, stream, log);
        if (e != hipSuccess) return e;
      }
    }
  }
  return hipSuccess;
}

// Host view of the launcher's plan for tests: the ranges the query axis (dK/dV kernel) or the key axis (dQ
// kernel) of a step is cut into, each with the piece description of its sub-mask and the block-mask offset.
int chunk_plan(const MaskDev& mk, int sq, int sk, bool query_axis, int max_ranges, int64_t* out) {
  const std::vector<RowRange> ranges = query_axis ? chunk_ranges(mk.q_nseg, mk.q_seg_len, sq, mk.blk ? mk.blk_q : 0)
                                                  : chunk_ranges(mk.k_nseg, mk.k_seg_len, sk, mk.blk ? mk.blk_k : 0);
  int n = 0;
  for (const RowRange& rg : ranges) {
    if (n == max_ranges) break;
    const MaskDev m = ranges.size() > 1 ? (query_axis ? sub_mask<true>(mk, rg.r0, rg.r1) : sub_mask<false>(mk, rg.r0, rg.r1)) : mk;
    int64_t* o = out + 7 * n++;
    o[0] = rg.r0;
    o[1] = rg.r1;
    o[2] = query_axis ? m.q_nseg : m.k_nseg;
    o[3] = query_axis ? m.q_seg_len : m.k_seg_len;
    o[4] = query_axis ? m.q_pos0 : m.k_pos0;
    o[5] = query_axis ? m.q_period : m.k_period;
    o[6] = m.blk ? (int64_t)(m.blk - mk.blk) : 0;
  }
  return (int)ranges.size();
}

hipError_t launch_steps_bwd(const BwdParams& p, const BwdStep* steps, int n, hipStream_t stream, LaunchLog* log) {
  if (p.head_dim == 128) return launch_bwd_groups<128>(p, steps, n, stream, log);
  return launch_bwd_groups<64>(p, steps, n, stream, log);
}

}  // namespace burst
