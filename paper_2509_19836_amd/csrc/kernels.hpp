// Kernel parameter blocks and host-side launchers shared between the C-ABI layer and the kernels.
#pragma once
#include <algorithm>
#include <vector>

#include "../../include/burst_attn_diag.h"
#include "common.hpp"

namespace burst {

// Rows may keep a stale running maximum until one of the wave's rows grows by more than
// 2^kLazyLog2; exp2 arguments then stay <= kLazyLog2, far inside fp32 / bf16 range.
constexpr float kLazyLog2 = 6.0f;

#ifndef BURST_A16
#define BURST_A16 4   // 16x16x32 streams, operands (two MFMAs each) ahead: 3 and 4 alike, 5 and 6 one to four percent slower
#endif
constexpr int kAhead16 = BURST_A16;

// What a launch walks: the key/value chunks of up to kMaxSteps ring steps of one query chunk, one after the other (a step
// whose key axis is cut into ranges is one for each).  All have the same query side; only a single one may have a
// block mask.
constexpr int kMaxSteps = 8;
struct FwdStep {
  MaskDev mask;
  int32_t sk;
  TensorDev k, v;
};

struct FwdParams {
  int32_t batch, q_heads, kv_heads, head_dim;
  int32_t sq, n_steps;
  float scale;
  TileRuns q_runs;      // query tiles with work, and the order of the work-groups (filled by the launcher)
  int32_t q_side_by_side;
  TensorDev q;
  TensorDev o_part;     // ptr == nullptr: not requested
  RowvecDev lse_part;
  TensorDev o_acc;      // ptr == nullptr: no fused merge
  RowvecDev lse_acc;
  FwdStep step[kMaxSteps];
};

struct BwdStep {
  MaskDev mask;
  int32_t sk;
  TensorDev k, v, dk, dv;   // dk, dv: fp32; ptr == nullptr: skip
  TileRuns k_runs;          // key tiles with work, the order of the work-groups and the first of them (filled by the launcher)
  int32_t k_side_by_side, first_block;
};

struct BwdParams {
  int32_t batch, q_heads, kv_heads, head_dim;
  int32_t sq, n_steps;
  float scale;
  TileRuns q_runs;          // query tiles with work, and the order of the work-groups (filled by the launcher)
  int32_t q_side_by_side;
  TensorDev q, d_o;
  RowvecDev lse, d;
  TensorDev dq;             // fp32; ptr == nullptr: skip
  int32_t acc_dq, acc_dk, acc_dv;
  BwdStep step[kMaxSteps];
};

struct MergeParams {
  int32_t batch, q_heads, head_dim, sq;
  TensorDev o_acc, o_part, o_out;   // o_out.ptr may be nullptr
  RowvecDev lse_acc, lse_part;
};

struct PreParams {
  int32_t batch, q_heads, head_dim, sq;
  TensorDev o, d_o;
  RowvecDev d;
};

// Runs of tiles, of `n`, for which nonempty(tile) holds.
template <class Nonempty>
inline TileRuns tile_runs(int n, Nonempty&& nonempty) {
  TileRuns tr{{0, 0}, {0, 0}};
  int nruns = 0;
  bool in_run = false;
  for (int t = 0; t < n; ++t) {
    if (!nonempty(t)) {
      in_run = false;
      continue;
    }
    if (!in_run) {
      if (nruns == 2) return TileRuns{{0, 0}, {n, 0}};   // more than two runs: launch every tile
      tr.start[nruns++] = t;
      in_run = true;
    }
    ++tr.len[nruns - 1];
  }
  return tr;
}
// Query tiles that see something of any of the steps' key chunks; key tiles of which the query chunk sees something.  The
// same classification the kernels use.
template <class Step>
inline TileRuns nonempty_q_runs(const Step* steps, int n_steps, int sq, int tile_rows) {
  return tile_runs((sq + tile_rows - 1) / tile_rows, [&](int t) {
    const int r0 = t * tile_rows, r1 = r0 + tile_rows < sq ? r0 + tile_rows : sq;
    for (int i = 0; i < n_steps; ++i)
      if (classify(steps[i].mask, r0, r1, 0, steps[i].sk, false) != TILE_SKIP) return true;
    return false;
  });
}
inline TileRuns nonempty_k_runs(const MaskDev& mk, int sq, int sk, int tile_rows) {
  return tile_runs((sk + tile_rows - 1) / tile_rows, [&](int t) {
    const int r0 = t * tile_rows, r1 = r0 + tile_rows < sk ? r0 + tile_rows : sk;
    return classify(mk, 0, sq, r0, r1, false) != TILE_SKIP;
  });
}

// Walk of the tile that is launched first (heaviest first: map_block) or last, in tiles of 64 rows of the other axis.
inline int q_tile_walk(const MaskDev& mk, int sq, int sk, int tile, int tile_rows) {
  const int end = tile * tile_rows + tile_rows;
  int lo, hi;
  range_minmax<true>(mk, tile * tile_rows, end < sq ? end : sq, lo, hi);
  return visible_tiles<false, 64>(mk, lo, hi, sk).len;
}
inline int k_tile_walk(const MaskDev& mk, int sq, int sk, int tile, int tile_rows) {
  const int end = tile * tile_rows + tile_rows;
  int lo, hi;
  range_minmax<false>(mk, tile * tile_rows, end < sk ? end : sk, lo, hi);
  return visible_tiles<true, 64>(mk, lo, hi, sq).len;
}
// A launch's tiles of one axis that see something: how many, about the sum of their walks, and about the longest one.  From up to
// eight of them, the first and the last one and some between at places that no regular pattern of walks repeats: two at the ends
// would stand for none where only rows in the middle see something, as against the shard one place ahead under the zigzag split with a window,
// and for half of the work under a window, whose walks are all alike but the first few.  (A block mask is not looked at.)
struct Walks {
  int64_t tiles, total, longest;
};
template <class Walk>
inline Walks sample_walks(int first, int end, bool alike, Walk&& walk) {
  constexpr int S = 8, at[S] = {0, 158, 61, 219, 37, 195, 98, 255};   // of 256, in an eighth of the tiles each; mirrored, so that walks that grow evenly average exactly
  const int64_t n = std::max(end - first, 0), s = alike ? std::min<int64_t>(n, 1) : std::min<int64_t>(n, S);
  Walks w{n, 0, 0};
  for (int i = 0; i < s; ++i) {
    const int64_t t = n <= S ? i : i == S - 1 ? n - 1 : (256 * i + at[i]) * n / (256 * S);
    const int64_t len = walk(first + (int)t);
    w.total += len;
    w.longest = std::max(w.longest, len);
  }
  if (s > 0) w.total = w.total * n / s;
  return w;
}
template <class Step>
inline Walks q_walks(const Step* steps, int n_steps, int sq, int tile_rows) {
  int lo = sq, hi = 0;
  bool alike = true;
  for (int i = 0; i < n_steps; ++i) {
    int olo, ohi;
    range_minmax<false>(steps[i].mask, 0, steps[i].sk, olo, ohi);
    const RowIntervals iv = row_intervals<true>(steps[i].mask, olo, ohi, sq, false);
    if (iv.some_lo >= iv.some_hi) continue;
    lo = std::min(lo, iv.some_lo);
    hi = std::max(hi, iv.some_hi);
    alike = alike && !steps[i].mask.causal;
  }
  return sample_walks(lo / tile_rows, (hi + tile_rows - 1) / tile_rows, alike, [&](int t) {
    int64_t len = 0;
    for (int i = 0; i < n_steps; ++i) len += q_tile_walk(steps[i].mask, sq, steps[i].sk, t, tile_rows);
    return len;
  });
}
inline Walks k_walks(const MaskDev& mk, int sq, int sk, int tile_rows) {
  int olo, ohi;
  range_minmax<true>(mk, 0, sq, olo, ohi);
  const RowIntervals iv = row_intervals<false>(mk, olo, ohi, sk, false);
  const int end = iv.some_lo < iv.some_hi ? (iv.some_hi + tile_rows - 1) / tile_rows : 0;
  return sample_walks(iv.some_lo / tile_rows, end, !mk.causal, [&](int t) { return (int64_t)k_tile_walk(mk, sq, sk, t, tile_rows); });
}
// Whether the walk of the tile that is launched last is at most half as long as that of the first one.
template <class Step>
inline bool uneven_q_walks(const Step* steps, int n_steps, int sq, const TileRuns& runs, int tile_rows) {
  const int n = runs.total();
  int first = 0, last = 0;
  for (int i = 0; i < n_steps && n > 0; ++i) {
    first += q_tile_walk(steps[i].mask, sq, steps[i].sk, runs.tile_of(n - 1), tile_rows);
    last += q_tile_walk(steps[i].mask, sq, steps[i].sk, runs.tile_of(0), tile_rows);
  }
  return n > 0 && 2 * last <= first;
}
inline bool uneven_k_walks(const MaskDev& mk, int sq, int sk, const TileRuns& runs, int tile_rows) {
  const int n = runs.total();
  return n > 0 && 2 * k_tile_walk(mk, sq, sk, runs.tile_of(n - 1), tile_rows) <= k_tile_walk(mk, sq, sk, runs.tile_of(0), tile_rows);
}
// About the longest walk of a step's query tiles of 256 rows, or key tiles of 128: of the first, the middle and the last one.
inline int longest_q_walk(const MaskDev& mk, int sq, int sk) {
  const int n = (sq + 255) / 256;
  return std::max({q_tile_walk(mk, sq, sk, 0, 256), q_tile_walk(mk, sq, sk, n / 2, 256), q_tile_walk(mk, sq, sk, n - 1, 256)});
}
inline int longest_k_walk(const MaskDev& mk, int sq, int sk) {
  const int n = (sk + 127) / 128;
  return std::max({k_tile_walk(mk, sq, sk, 0, 128), k_tile_walk(mk, sq, sk, n / 2, 128), k_tile_walk(mk, sq, sk, n - 1, 128)});
}
// Whether a launch runs the keys of an XCD (of two or more) side by side (map_block).  A block mask makes any walks uneven.
template <class Step>
inline bool q_side_by_side(const Step* steps, int n_steps, int sq, int n_keys, int group, const TileRuns& runs, int tile_rows) {
  return n_keys >= 16 && short_launch(n_keys, group, runs.total()) &&
         (steps[0].mask.blk || uneven_q_walks(steps, n_steps, sq, runs, tile_rows));
}
inline bool k_side_by_side(const MaskDev& mk, int sq, int sk, int n_keys, const TileRuns& runs, int tile_rows) {
  return n_keys >= 16 && short_launch(n_keys, 1, runs.total()) && (mk.blk || uneven_k_walks(mk, sq, sk, runs, tile_rows));
}

// ---------------------------------------------------------------------------------------------
// Chunked launches.  The work-groups that share an XCD's L2 (4 MiB) walk the streamed axis side by side,
// so a tile of it is fetched from HBM about once -- as long as the walk is short enough for them to stay
// together.  Over a walk of thousands of tiles they drift apart and each streams its own copy (at 131072-row
// chunks the dQ kernel fetched 107 GB per step instead of 32 GB).  A long streamed axis is therefore cut into
// row ranges of about chunk_rows() rows, one launch per range on the same stream, the stationary side's
// result accumulating in HBM from launch to launch (dQ; dK and dV; the forward kernel's running O and Lse,
// when the step result itself is not asked for).  Ranges of 32768 rows cost no time (16384: 1 %, 8192: 4 %).
// A range lies inside one piece of the axis or covers whole pieces, so it is again a chunk the mask
// descriptor can express.
int chunk_rows();   // the range length in force (set_chunk_rows; api.hip holds the value)

struct RowRange {
  int r0, r1;
};
// Ranges that cover [0, rows) of an axis of nseg pieces of seg_len rows; one range (no chunking) when the
// axis is short or a block mask's row blocks would be cut.
inline std::vector<RowRange> chunk_ranges(int nseg, int seg_len, int rows, int blk_rows) {
  const int target = chunk_rows();
  std::vector<RowRange> out;
  const bool cuts_blocks = blk_rows > 0 && ((nseg > 1 && seg_len % blk_rows != 0) || target % blk_rows != 0);
  if (rows <= 2 * target || cuts_blocks) {
    out.push_back({0, rows});
    return out;
  }
  if (nseg <= 1 || seg_len >= target) {   // ranges inside each piece
    const int pieces = nseg <= 1 ? 1 : nseg, len = nseg <= 1 ? rows : seg_len;
    for (int s = 0; s < pieces; ++s)
      for (int a = 0; a < len; a += target) out.push_back({s * len + a, s * len + (a + target < len ? a + target : len)});
  } else {                                // whole pieces per range
    const int per = target / seg_len > 0 ? target / seg_len : 1;
    for (int s = 0; s < nseg; s += per) out.push_back({s * seg_len, (s + per < nseg ? s + per : nseg) * seg_len});
  }
  return out;
}
// The mask of rows [r0, r1) of the query axis (Q_AXIS) or the key axis against the whole other axis.
template <bool Q_AXIS>
inline MaskDev sub_mask(const MaskDev& mk, int r0, int r1) {
  MaskDev m = mk;
  int32_t& nseg = Q_AXIS ? m.q_nseg : m.k_nseg;
  int32_t& seg_len = Q_AXIS ? m.q_seg_len : m.k_seg_len;
  int32_t& pos0 = Q_AXIS ? m.q_pos0 : m.k_pos0;
  int32_t& period = Q_AXIS ? m.q_period : m.k_period;
  if (nseg <= 1) {
    pos0 += r0 * m.pos_stride;
    seg_len = r1 - r0;
  } else {
    const int s0 = r0 / seg_len;
    if ((r1 - 1) / seg_len == s0) {   // inside piece s0
      pos0 += s0 * period + (r0 - s0 * seg_len) * m.pos_stride;
      nseg = 1;
      period = 0;
      seg_len = r1 - r0;
    } else {                          // pieces s0 .. (r1 / seg_len) - 1, whole
      pos0 += s0 * period;
      nseg = (r1 - r0) / seg_len;
    }
  }
  if (m.blk) m.blk += Q_AXIS ? (int64_t)(r0 / m.blk_q) * m.blk_pitch : (int64_t)(r0 / m.blk_k);
  return m;
}
inline void offset_rows(TensorDev& t, int r0) { t.ptr = (char*)t.ptr + (int64_t)r0 * t.ss * (t.is_f32 ? 4 : 2); }

// Steps that one launch walks.  Consecutive steps of a ring whose shards are all there share a launch (they have the same
// query side): a query tile keeps its state in registers from shard to shard, and there is one last, part-empty round of
// work-groups instead of one for each.  A ring, d = 128, us step by step and shared: 8 shards of 8192 rows, 16/2 heads:
// forward 1826, 1706, dQ 2500, 2357, dK/dV 5446, 3657; 4 shards of 4096 rows, 32 heads: dQ 696, 613, dK/dV 1003, 961; 4
// of 1500 rows, 48 heads, d = 64: forward 181, 160, dQ 195, 176, dK/dV 238, 193; 4 of 8192 rows, 32 heads: 1891, 1823, 2542, 2427,
// 3621, 3579.  Beyond kShareLaunch tiles of 256 rows a step (4 per CU; key tiles of 128 rows are twice as many) there is
// nothing to gain: 8 shards of 16384 rows, 32 heads, zigzag: forward 13753, 13778, dQ 18904, 18828, dK/dV 26695, 27106,
// striped: 14816, 15190, 20535, 20615, 29172, 29317.
// Walks of up to kShareWalk tiles are short enough for what every step costs beside its tiles (the first loads, O or dQ read and
// written) to count however many there are.  us step by step and shared, forward and dQ: 8 shards of 16384 rows, 32 heads, striped, with
// a window of 4000 tokens (12 tiles a step) 2446, 1830 and 2801, 2104; of 12000 (28) 3934, 3390 and 4897, 4440; of 32768 (68) 7213, 6931 and
// 9464, 9076; of 65536 (132) 11125, 11091 and 14923, 14842; 8 of 4096 rows, 2 x 64/8 heads (64) 3857, 3417 and 5201, 4678; 4 of 3000, 8 x
// 16 (47) 1927, 1768 and 2557, 2398; 4 of 8000, 64 (125) 3679, 3836 and 4905, 5186.  Key tiles up to kShareKeyWalk: dK/dV with the window of 1000
// (6 tiles) 3008, 2819; 4000 (10) 3940, 3763; 12000 6730, 6622; 32768 13049, 13130; at d = 64 8 x 16 x 3000 (47) 2030, 2046-2110.
// A step with a block mask goes alone, and the walks of these launches together are bounded by what stays in step in an L2, two
// ranges.  Not so in the joint backward launch (launch_both_t), which takes up to kMaxSteps chunks of a range each: 1
// head, 8 shards of 32768 rows, backward in calls of 1, 2 and 8 steps: full 13.42, 11.61, 11.53 ms, zigzag 9.02, 6.69, 6.87, striped
// 11.62, 7.99, 8.87.  Steps of which no query row sees anything are left out.  launch(first, end): steps [first, end) of `parts`.
constexpr int kShareLaunch = 1024, kShareWalk = 80, kShareKeyWalk = 40;
inline bool share_launch(int heads, int rows) { return (int64_t)heads * ((rows + 255) / 256) <= kShareLaunch; }
template <class Step, class Launch>
inline hipError_t for_step_groups(std::vector<Step>& parts, int sq, int heads, Launch&& launch) {
  parts.erase(std::remove_if(parts.begin(), parts.end(),
                             [&](const Step& st) { return classify(st.mask, 0, sq, 0, st.sk, false) == TILE_SKIP; }), parts.end());
  const int n = (int)parts.size();
  const bool share = share_launch(heads, sq);
  for (int first = 0, end = 0; first < n; first = end) {
    int64_t rows = 0;
    bool all = true;   // so far, walks short enough for the others to join
    for (; end < n; ++end) {
      const int walk = n > 1 ? longest_q_walk(parts[end].mask, sq, parts[end].sk) : 0;
      all = all && (share || walk <= kShareWalk);
      if (end > first && (!all || parts[end].mask.blk || parts[first].mask.blk || end - first == kMaxSteps ||
                          rows + 64ll * walk > 2ll * chunk_rows()))
        break;
      rows += 64ll * walk;
    }
    const hipError_t e = launch(first, end);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Fused LM head + cross-entropy (Alg. 3).  Sizes are validated on the host; the workspace is carved up there.
struct LmHeadParams {
  int32_t n_tokens, d_model, vocab, tile_tokens;
  int32_t v_pad;        // vocab rounded up to 256: row length of the two workspace matrices
  float grad_scale;
  const __bf16* h;      // [n_tokens][ld_h]
  const __bf16* w;      // [vocab][ld_w]
  int64_t ld_h, ld_w;
  const int64_t* y;
  float* loss;
  float* lse;           // may be nullptr
  void* dh;             // may be nullptr
  int32_t dh_is_f32;
  int64_t ld_dh;
  float* dw;            // may be nullptr
  int64_t ld_dw;
  int32_t acc_dw;
  float* logits;        // workspace [tile_tokens][v_pad]
  __bf16* dlogits;      // workspace [tile_tokens][v_pad]
  float2* part;         // workspace [v_pad / 128][tile_tokens]: (max, sum of exp) over 128 words
  __bf16* ht;           // workspace [d_model][tile_tokens]: the sequence tile's rows of h, transposed
};
int64_t lm_head_workspace_bytes(int64_t tile_tokens, int64_t vocab, int64_t d_model);
void lm_head_tile_plan(const LmHeadParams& p, int32_t out[6]);   // burst_lm_head_tile_plan, from the sizes in p
hipError_t launch_lm_head_loss(const LmHeadParams& p, hipStream_t stream);

// n steps of the query chunk that `p` describes (its own step array is not read).  More than one only without o_part.
// With a log nothing is launched: it gets the kernel (BURST_KERNEL_ bits) of each launch of step kernels that there would be.
typedef std::vector<int32_t> LaunchLog;
hipError_t launch_steps_fwd(const FwdParams& p, const FwdStep* steps, int n, hipStream_t stream, LaunchLog* log = nullptr);
hipError_t launch_steps_bwd(const BwdParams& p, const BwdStep* steps, int n, hipStream_t stream, LaunchLog* log = nullptr);
// rows of the streamed axis per launch of a step kernel (longer axes are cut into several launches)
void set_chunk_rows(int rows);
int chunk_plan(const MaskDev& mk, int sq, int sk, bool query_axis, int max_ranges, int64_t* out);
hipError_t launch_lse_merge(const MergeParams& p, hipStream_t stream);
hipError_t launch_preprocess_bwd(const PreParams& p, hipStream_t stream);
// o_part = 0 / lse_part = -inf for a step with no key rows; zero-fill of fp32 gradients
hipError_t launch_fill_empty_fwd(const FwdParams& p, hipStream_t stream);
hipError_t launch_mfma_probe(float* sink, int iters, int random_operands, int64_t* flops, hipStream_t stream);
hipError_t launch_zero_tensor(const TensorDev& t, int32_t batch, int32_t rows, int32_t heads, int32_t head_dim,
                              hipStream_t stream);

}  // namespace burst
