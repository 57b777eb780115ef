"""Edges of the work-group mapping and of the tile pipelines.

Head and batch counts that do not fill whole rounds of the eight XCDs: the work-group mapping deals the
left-over (batch, kv head) keys tile by tile over all XCDs, and long launches walk an XCD's keys one after the
other where short ones run them side by side.  Every work-group owns its outputs, so a tile that the mapping
dropped or dealt twice to different heads shows as a wrong element against the oracle."""
import numpy as np
import pytest

from oracle import burst_oracle as oc
from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def step_case(lib, B, Hq, Hkv, d, sq, sk, causal, seed, q_pos=0, k_pos=0):
    """One forward step (step result) and one backward step (overwriting) against the oracle, every element."""
    import torch
    rng = np.random.Generator(np.random.PCG64(wl.BASE_SEED + 61000 + seed))
    desc = f"B={B} heads={Hq}/{Hkv} d={d} sq={sq}@{q_pos} sk={sk}@{k_pos} causal={causal}"
    print(desc, flush=True)
    draw = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    qb, kb, vb, gb = draw(B, sq, Hq, d), draw(B, sk, Hkv, d), draw(B, sk, Hkv, d), draw(B, sq, Hq, d)
    Q, K, V, G = (hp.widen(x) for x in (qb, kb, vb, gb))
    q, k, v, g = (hp.dev_bf16(x) for x in (qb, kb, vb, gb))
    mask = lib.burst_mask_t()
    mask.mode = lib.BURST_MASK_CAUSAL if causal else lib.BURST_MASK_FULL
    mask.q_nseg = mask.k_nseg = mask.pos_stride = 1
    mask.q_seg_len, mask.k_seg_len = sq, sk
    mask.q_seg_pos[0], mask.k_seg_pos[0] = q_pos, k_pos
    vis = oc.visibility(q_pos + np.arange(sq), k_pos + np.arange(sk), causal)
    scale = 1.0 / float(np.sqrt(d))
    shp = lib.shape(B, Hq, Hkv, d, sq, sk, scale)
    O_ref, lse_ref = oc.mha_step_fwd(Q, K, V, scale, vis)
    nan = lambda *shape: torch.full(shape, float("nan"), device="cuda", dtype=torch.float32)
    o, lse = nan(B, sq, Hq, d), nan(B, Hq, sq)
    lib.burst_attn_step_fwd(shp, mask, q, k, v, o_part=o, lse_part=lse)
    torch.cuda.synchronize()
    assert hp.rel_err(o.cpu().numpy(), O_ref) <= hp.REL_TOL, desc
    assert hp.lse_err(lse.cpu().numpy(), lse_ref) <= hp.LSE_TOL, desc
    lse_in = np.where(np.isfinite(lse_ref), lse_ref, 0.0).astype(np.float32) + np.float32(0.25)
    D_in = rng.standard_normal((B, Hq, sq)).astype(np.float32)
    ref = oc.mha_step_bwd(Q, K, V, G, lse_in.astype(np.float64), D_in.astype(np.float64), scale, vis)
    out = nan(B, sq, Hq, d), nan(B, sk, Hkv, d), nan(B, sk, Hkv, d)
    lib.burst_attn_step_bwd(shp, mask, q, k, v, g, torch.from_numpy(lse_in).cuda(), torch.from_numpy(D_in).cuda(),
                            dq=out[0], dk=out[1], dv=out[2])
    torch.cuda.synchronize()
    for name, got, want in zip(("dQ", "dK", "dV"), out, ref):
        assert hp.rel_err(got.cpu().numpy(), want) <= hp.REL_TOL, (name, desc)


@pytest.mark.parametrize("B,Hq,Hkv,d,n,causal", [
    (1, 1, 1, 64, 300, True),        # one key: tiles dealt over all XCDs
    (1, 6, 3, 128, 520, True),       # three keys, groups of two
    (1, 9, 9, 64, 260, False),       # one whole round and one key left over
    (5, 3, 3, 64, 513, True),        # fifteen keys over the batch
    (2, 28, 7, 128, 257, True),      # groups of four
    (8, 40, 5, 64, 1800, True),      # five whole rounds, groups of eight: more than a short launch
])
def test_head_layouts(lib, B, Hq, Hkv, d, n, causal):
    step_case(lib, B, Hq, Hkv, d, n, n, causal, B * 1000 + Hq)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("sk", [1, 63, 64, 65, 128, 192, 257, 320, 449])
def test_short_walks(lib, d, sk):
    """Key chunks of one to eight tiles, whole and ragged, under both masks: the pipelines fetch up to four tiles
    ahead, so every walk shorter than that has its own prologue and end; query rows that fill no wave."""
    step_case(lib, 1, 2, 2, d, 77, sk, False, sk)
    step_case(lib, 1, 2, 1, d, 300, sk, True, sk + 1, q_pos=40)


@pytest.mark.parametrize("B,H,d,sq,sk,causal", [
    (1, 1, 128, 33, 1, False),       # one key row
    (1, 3, 64, 97, 65, True),        # second key tile of one row; the second pair of a key block has one query row
    (2, 2, 128, 161, 191, True),     # pairs that see nothing of a tile
    (4, 32, 64, 130, 128, False),    # 128 tiles of 128: the last count that takes tiles of 64
    (4, 33, 64, 130, 128, False),    # 132: tiles of 128 where the walks are even,
    (3, 40, 128, 257, 257, True),    # 360: more than one per CU, tiles of 128
    (2, 40, 128, 200, 250, True),    # 160, uneven: tiles of 64
    (1, 256, 64, 190, 90, True),     # 256, one tile a head: even walks
])
def test_key_tile_heights(lib, B, H, d, sq, sk, causal):
    """The dK/dV kernel's two key tile heights, at the counts where the launcher changes from one to the other."""
    step_case(lib, B, H, H, d, sq, sk, causal, B * 1000 + H + sk)


@pytest.mark.parametrize("B,Hq,Hkv,d,sq,sk,causal", [
    (1, 1, 1, 64, 1, 1, True),
    (1, 4, 2, 128, 300, 191, True),    # key tiles of 64
    (2, 33, 33, 64, 259, 333, False),  # key tiles of 128, work-groups of all eight XCDs in both parts
    (1, 2, 2, 128, 700, 1100, True),   # key tiles that see nothing: zeros are written before the launch
])
def test_gradients_together_and_apart(lib, B, Hq, Hkv, d, sq, sk, causal):
    """A short step computes dQ and dK/dV in one launch; asked for one by one they take a launch each.  The order of
    every sum is the same; 1e-6 of the largest entry is left for the compiler's contraction of products and sums."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(wl.BASE_SEED + sq + sk)
    f32 = dict(device="cuda", dtype=torch.float32)
    draw = lambda *shape: torch.randn(*shape, generator=gen, **f32)
    q, g = (draw(B, sq, Hq, d).to(torch.bfloat16) for _ in range(2))
    k, v = (draw(B, sk, Hkv, d).to(torch.bfloat16) for _ in range(2))
    lse, D = 5 + draw(B, Hq, sq), draw(B, Hq, sq)
    mask = lib.burst_mask_t()
    mask.mode = lib.BURST_MASK_CAUSAL if causal else lib.BURST_MASK_FULL
    mask.q_nseg = mask.k_nseg = mask.pos_stride = 1
    mask.q_seg_len, mask.k_seg_len = sq, sk
    shp = lib.shape(B, Hq, Hkv, d, sq, sk, d ** -0.5)
    for flags in (0, lib.BURST_ACC_DQ | lib.BURST_ACC_DK | lib.BURST_ACC_DV):
        both, apart = ([torch.full(x.shape, 0.5 if flags else float("nan"), **f32) for x in (q, k, v)] for _ in range(2))
        print(f"together / apart B={B} {Hq}/{Hkv} d={d} {sq}x{sk} causal={causal} flags={flags}", flush=True)
        lib.burst_attn_step_bwd(shp, mask, q, k, v, g, lse, D, dq=both[0], dk=both[1], dv=both[2], accumulate_flags=flags)
        lib.burst_attn_step_bwd(shp, mask, q, k, v, g, lse, D, dq=apart[0], accumulate_flags=flags)
        lib.burst_attn_step_bwd(shp, mask, q, k, v, g, lse, D, dk=apart[1], dv=apart[2], accumulate_flags=flags)
        torch.cuda.synchronize()
        for name, x, y in zip(("dQ", "dK", "dV"), both, apart):
            assert (x - y).abs().max() <= 1e-6 * y.abs().max(), (name, flags)


@pytest.mark.parametrize("B,Hq,Hkv,d,sq,sk,causal,q_pos", [
    (2, 16, 8, 64, 800, 800, True, 0),       # uneven walks: the keys of an XCD side by side
    (2, 16, 8, 64, 800, 800, False, 0),      # all walks alike: one after the other
    (1, 19, 19, 128, 530, 700, True, 700),   # an earlier shard: alike, three keys left over
    (1, 19, 19, 128, 700, 530, True, 100),   # some tiles without keys, uneven
    (1, 48, 16, 64, 700, 300, True, 200),    # even for the queries' tiles, uneven for the keys'
])
def test_order_of_the_keys_of_an_xcd(lib, B, Hq, Hkv, d, sq, sk, causal, q_pos):
    step_case(lib, B, Hq, Hkv, d, sq, sk, causal, B * 1000 + Hq + sq, q_pos=q_pos)
