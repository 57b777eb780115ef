"""Block masks with long runs of closed tiles: the cursors of all three kernels find the open ones 64 tiles at a time.

Runs of exactly 64 tiles, of 64 to 128 and of more than 128, at the start of a walk and inside it, behind which an open
tile, the ragged last one or nothing follows; two query heads to a key head, so that a walk starts over."""
import numpy as np
import pytest

from oracle import burst_oracle as oc
from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu

LONG, B, Hq, Hkv = 9000, 1, 2, 1   # 141 tiles of 64 rows, the last one of 40


def _pattern(lines, blocks, block_tiles):
    """lines x blocks: line 0 has 64 closed tiles between two open blocks, 1 has 64 and more before the only open one,
    2 more than 128 between two, 3 the ragged last block alone, 4 nothing, 5 everything."""
    after = 64 // block_tiles
    open_at = [[0, 1 + after], [1 + after], [0, blocks - 2], [blocks - 1], [], range(blocks)]
    bm = np.zeros((lines, blocks), np.uint8)
    for line, at in enumerate(open_at):
        bm[line, list(at)] = 1
    return bm


def _mask(lib, causal, sq, sk):
    # causal: the walk of a query starts among the first keys, that of a key behind them
    return lib.burst_mask_t(int(causal), 1, 1, 0, (0 if sq == LONG else LONG - 1000, 0), (3000 if sq == LONG else 0, 0), sq, sk, 1)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("walk", ["queries", "keys"])
def test_walks_over_long_runs_of_closed_tiles(lib, walk, d, causal):
    import torch
    if walk == "queries":
        sq, sk, bq, bk = LONG, 5 * 128 + 40, 256, 128
        bm = _pattern(6, -(-sq // bq), 4).T
    else:
        sq, sk, bq, bk = 5 * 256 + 40, LONG, 256, 128
        bm = _pattern(6, -(-sk // bk), 2)
    rng = np.random.Generator(np.random.PCG64(wl.BASE_SEED + 73000 + d + sq))
    draw = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    qb, kb, vb, gb = draw(B, sq, Hq, d), draw(B, sk, Hkv, d), draw(B, sk, Hkv, d), draw(B, sq, Hq, d)
    Q, K, V, G = (hp.widen(x) for x in (qb, kb, vb, gb))
    mask = _mask(lib, causal, sq, sk)
    bm_dev = torch.from_numpy(np.ascontiguousarray(bm)).cuda()
    lib.set_block_mask(mask, bm_dev, bq, bk)
    vis = oc.apply_block_mask(oc.visibility(hp.mask_positions(mask, "q"), hp.mask_positions(mask, "k"), causal), bm, bq, bk)
    scale = d ** -0.5
    shp = lib.shape(B, Hq, Hkv, d, sq, sk, scale)
    q, k, v, g = (hp.dev_bf16(x) for x in (qb, kb, vb, gb))
    new = lambda *shape: torch.full(shape, float("nan"), device="cuda", dtype=torch.float32)
    O_ref, lse_ref = oc.mha_step_fwd(Q, K, V, scale, vis)
    o, lse = new(B, sq, Hq, d), new(B, Hq, sq)
    print(f"closed runs, {walk} d={d} causal={causal}", flush=True)
    lib.burst_attn_step_fwd(shp, mask, q, k, v, o_part=o, lse_part=lse)
    torch.cuda.synchronize()
    assert hp.rel_err(o.cpu().numpy(), O_ref) <= hp.REL_TOL
    assert hp.lse_err(lse.cpu().numpy(), lse_ref) <= hp.LSE_TOL
    lse_in = (np.where(np.isfinite(lse_ref), lse_ref, 0.0) + 0.25).astype(np.float32)
    D_in = rng.standard_normal((B, Hq, sq)).astype(np.float32)
    refs = oc.mha_step_bwd(Q, K, V, G, lse_in.astype(np.float64), D_in.astype(np.float64), scale, vis)
    dq, dk, dv = new(B, sq, Hq, d), new(B, sk, Hkv, d), new(B, sk, Hkv, d)
    lib.burst_attn_step_bwd(shp, mask, q, k, v, g, torch.from_numpy(lse_in).cuda(), torch.from_numpy(D_in).cuda(),
                            dq=dq, dk=dk, dv=dv)
    torch.cuda.synchronize()
    for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), refs):
        assert hp.rel_err(got.cpu().numpy(), ref) <= hp.REL_TOL, name
