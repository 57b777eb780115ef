"""Infinities and NaN in keys and values that a query row may not see stay away from it.

A wave owns 32 query rows and meets the keys in tiles of 64: rows whose group of 32 sees nothing of the tile that holds
a non-finite key or value give the result they give with finite numbers there, whatever the work-group's other rows see."""
import numpy as np
import pytest

from oracle import burst_oracle as oc
from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu

GROUP, TILE = 32, 64


def _mask(lib, kind):
    """(mask, sq, sk, poisoned key rows)"""
    m = lib.burst_mask_t()
    m.mode, m.pos_stride = lib.BURST_MASK_CAUSAL, 1
    m.q_nseg = m.k_nseg = 1
    if kind == "causal":            # later keys inside the work-group's own range
        m.q_seg_len = m.k_seg_len = 512
        return m, 512, 512, [170, 511]
    if kind == "window":            # keys that have left the window, and later ones
        m.q_seg_len = m.k_seg_len = 512
        m.window = 40
        return m, 512, 512, [0, 130, 400]
    if kind == "zigzag":            # two pieces a side that fit no tile
        m.q_nseg = m.k_nseg = 2
        m.q_seg_len = m.k_seg_len = 150
        m.q_seg_pos[:] = m.k_seg_pos[:] = (150, 600)
        return m, 300, 300, [140, 299]
    if kind == "left_behind":       # a ragged last key tile that the later rows' window has left altogether
        m.q_seg_len, m.k_seg_len = 256, 70
        m.q_seg_pos[0] = 60
        m.window = 30
        return m, 256, 70, [69]
    raise ValueError(kind)


@pytest.mark.parametrize("blocks", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["causal", "window", "zigzag", "left_behind"])
def test_rows_that_see_nothing_of_a_tile_are_not_touched_by_it(lib, kind, d, blocks):
    import torch
    mask, sq, sk, rows = _mask(lib, kind)
    B, Hq, Hkv = 1, 2, 1
    rng = np.random.Generator(np.random.PCG64(wl.BASE_SEED + 71000 + d))
    draw = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    qb, kb, vb, gb = draw(B, sq, Hq, d), draw(B, sk, Hkv, d), draw(B, sk, Hkv, d), draw(B, sq, Hq, d)
    Q, K, V, G = (hp.widen(x) for x in (qb, kb, vb, gb))
    vis = oc.visibility(hp.mask_positions(mask, "q"), hp.mask_positions(mask, "k"), True, mask.window)
    if blocks:
        bm = torch.ones((-(-sq // 256), -(-sk // 128)), dtype=torch.uint8, device="cuda")
        lib.set_block_mask(mask, bm, 256, 128)
    clean = np.ones(sq, bool)
    for row in rows:
        t0 = row // TILE * TILE
        for g0 in range(0, sq, GROUP):
            if vis[g0:g0 + GROUP, t0:t0 + TILE].any():
                clean[g0:g0 + GROUP] = False
    assert clean.any() and not clean.all()
    q, g = hp.dev_bf16(qb), hp.dev_bf16(gb)
    bad = lambda bits, value: (lambda t: (t.__setitem__((slice(None), rows), value), t)[1])(hp.dev_bf16(bits))
    shp = lib.shape(B, Hq, Hkv, d, sq, sk, d ** -0.5)
    O_ref, lse_ref = oc.mha_step_fwd(Q, K, V, d ** -0.5, vis)
    lse_in = np.where(np.isfinite(lse_ref), lse_ref, 0.0).astype(np.float32) + np.float32(0.25)
    D_in = rng.standard_normal((B, Hq, sq)).astype(np.float32)
    dQ_ref = oc.mha_step_bwd(Q, K, V, G, lse_in.astype(np.float64), D_in.astype(np.float64), d ** -0.5, vis)[0]
    new = lambda *shape: torch.zeros(shape, device="cuda", dtype=torch.float32)
    for value in (float("inf"), float("nan")):
        print(f"{kind} d={d} blocks={blocks} value={value}", flush=True)
        o, lse = new(B, sq, Hq, d), new(B, Hq, sq)
        lib.burst_attn_step_fwd(shp, mask, q, hp.dev_bf16(kb), bad(vb, value), o_part=o, lse_part=lse)
        torch.cuda.synchronize()
        assert hp.rel_err(o.cpu().numpy()[:, clean], O_ref[:, clean]) <= hp.REL_TOL
        assert hp.lse_err(lse.cpu().numpy()[:, :, clean], lse_ref[:, :, clean]) <= hp.LSE_TOL
        for alone in (True, False):   # the dQ launch, and the joint one of a short step
            dq = new(B, sq, Hq, d)
            rest = {} if alone else {"dk": new(B, sk, Hkv, d), "dv": new(B, sk, Hkv, d)}
            lib.burst_attn_step_bwd(shp, mask, q, bad(kb, value), hp.dev_bf16(vb), g, torch.from_numpy(lse_in).cuda(),
                                    torch.from_numpy(D_in).cuda(), dq=dq, **rest)
            torch.cuda.synchronize()
            assert hp.rel_err(dq.cpu().numpy()[:, clean], dQ_ref[:, clean]) <= hp.REL_TOL, alone
