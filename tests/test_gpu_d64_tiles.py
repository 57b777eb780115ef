"""Edges of the tiles of the 64-wide heads' kernels: work-groups of 128 query rows with three tiles of 64 rows in LDS.

One row to a row more than a tile on either side, one tile to one more than there are in LDS, waves without rows, the diagonal
of a causal mask through a tile.  (Launches as small as test_tiles_of_narrow_heads' deal their walks to the waves of
a work-group; test_gpu_whole_walks.py runs it again on the kernels of three tiles in LDS.)"""
import pytest

from tests.test_gpu_head_layouts import step_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("sq,sk", [(1, 1), (1, 257), (31, 64), (33, 65), (127, 128), (128, 129), (129, 192), (160, 193), (255, 320), (385, 63)])
def test_tiles_of_narrow_heads(lib, sq, sk, causal):
    step_case(lib, 1, 6, 3, 64, sq, sk, causal, 500 + sq + sk, q_pos=40)


@pytest.mark.parametrize("sq,sk,causal,window", [(513, 513, False, 0), (640, 577, True, 0), (500, 700, True, 130), (129, 1025, False, 0)])
@pytest.mark.parametrize("blocks", [False, True])
def test_work_groups_that_share_a_cu(lib, sq, sk, causal, window, blocks):
    """Gradients of enough heads for several work-groups per CU: all in one call, dQ alone, dK and dV alone."""
    import numpy as np
    import torch
    from oracle import burst_oracle as oc
    from paper_2509_19836_amd import workloads as wl
    from tests import helpers as hp
    B, Hq, Hkv, d = 8, 24, 12, 64
    rng = np.random.Generator(np.random.PCG64(wl.BASE_SEED + 73000 + sq + sk))
    draw = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    qb, kb, vb, gb = draw(B, sq, Hq, d), draw(B, sk, Hkv, d), draw(B, sk, Hkv, d), draw(B, sq, Hq, d)
    mask = lib.burst_mask_t()
    mask.mode = lib.BURST_MASK_CAUSAL if causal else lib.BURST_MASK_FULL
    mask.q_nseg = mask.k_nseg = mask.pos_stride = 1
    mask.q_seg_len, mask.k_seg_len, mask.window = sq, sk, window
    q_pos = 150 if causal else 0
    mask.q_seg_pos[0] = q_pos
    vis = oc.visibility(q_pos + np.arange(sq), np.arange(sk), causal, window)
    if blocks:
        bm = rng.integers(0, 2, (-(-sq // 256), -(-sk // 128))).astype(np.uint8)
        bm[0, 0] = 1
        on_gpu = torch.from_numpy(bm).cuda()
        lib.set_block_mask(mask, on_gpu, 256, 128)
        vis = (np.ones((sq, sk), bool) if vis is None else vis) & (np.kron(bm, np.ones((256, 128), np.uint8))[:sq, :sk] != 0)
    scale = d ** -0.5
    lse = rng.normal(3.0, 0.3, (B, Hq, sq)).astype(np.float32)
    D = rng.standard_normal((B, Hq, sq)).astype(np.float32)
    ref = oc.mha_step_bwd(*(hp.widen(x) for x in (qb, kb, vb, gb)), lse.astype(np.float64), D.astype(np.float64), scale, vis)
    q, k, v, g = (hp.dev_bf16(x) for x in (qb, kb, vb, gb))
    shp = lib.shape(B, Hq, Hkv, d, sq, sk, scale)
    nan = lambda *shape: torch.full(shape, float("nan"), device="cuda", dtype=torch.float32)
    for want in ("dQ dK dV", "dQ", "dK dV"):
        out = {n: nan(B, sq, Hq, d) if n == "dQ" else nan(B, sk, Hkv, d) for n in want.split()}
        print(sq, sk, causal, window, blocks, want, flush=True)
        lib.burst_attn_step_bwd(shp, mask, q, k, v, g, torch.from_numpy(lse).cuda(), torch.from_numpy(D).cuda(),
                                **{n.lower(): t for n, t in out.items()})
        torch.cuda.synchronize()
        for n, r in zip(("dQ", "dK", "dV"), ref):
            if n in out:
                assert hp.rel_err(out[n].cpu().numpy(), r) <= hp.REL_TOL, (n, want)


@pytest.mark.parametrize("B,Hq,Hkv,sq,sks,causal", [
    (2, 32, 8, 1000, (1000,), False),
    (2, 32, 8, 700, (961,), False),          # a last key tile of one row
    (2, 32, 8, 1025, (897,), False),         # a last query tile of one row
    (1, 64, 8, 1000, (961, 1000), False),    # two steps
    (2, 64, 8, 1000, (1000, 961), True),     # and walks of any length
])
def test_work_groups_that_share_a_cu_with_key_tiles_of_64(lib, B, Hq, Hkv, sq, sks, causal):
    """The joint launch with few key tiles and long walks over grouped heads: two pairs of waves share 32 key rows and add their
    sums up in LDS beside the three tiles there.  Behind the rows of every input stands NaN."""
    import numpy as np
    import torch
    from oracle import burst_oracle as oc
    from paper_2509_19836_amd import workloads as wl
    from tests import helpers as hp
    d, scale = 64, 0.125
    rng = np.random.Generator(np.random.PCG64(wl.BASE_SEED + 74000 + sq + sum(sks)))
    draw = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    qb, gb = draw(B, sq, Hq, d), draw(B, sq, Hq, d)
    kv = [(draw(B, sk, Hkv, d), draw(B, sk, Hkv, d)) for sk in sks]
    masks, seen, at = [], [], 0
    for sk in sks:
        m = lib.burst_mask_t()
        m.mode = lib.BURST_MASK_CAUSAL if causal else lib.BURST_MASK_FULL
        m.q_nseg = m.k_nseg = m.pos_stride = 1
        m.q_seg_len, m.k_seg_len = sq, sk
        m.q_seg_pos[0], m.k_seg_pos[0] = 1000, at
        seen.append(oc.visibility(1000 + np.arange(sq), at + np.arange(sk), causal))
        masks.append(m)
        at += sk
    shapes = [lib.shape(B, Hq, Hkv, d, sq, sk, scale) for sk in sks]
    assert lib.burst_attn_launch_plan("bwd", shapes, masks) == [
        lib.BURST_KERNEL_DQ | lib.BURST_KERNEL_DKDV | lib.BURST_KERNEL_SHARED_CU | lib.BURST_KERNEL_KEY_TILES_64]
    lse = rng.normal(6.0, 0.3, (B, Hq, sq)).astype(np.float32)
    D = rng.standard_normal((B, Hq, sq)).astype(np.float32)
    Q, G = hp.widen(qb), hp.widen(gb)
    refs = [oc.mha_step_bwd(Q, hp.widen(kb), hp.widen(vb), G, lse.astype(np.float64), D.astype(np.float64), scale, vis)
            for (kb, vb), vis in zip(kv, seen)]

    def padded(x, axis):
        pad = list(x.shape)
        pad[axis] = 70
        return torch.cat([x, torch.full(pad, float("nan"), device="cuda", dtype=x.dtype)], axis).narrow(axis, 0, x.shape[axis])
    q, g = padded(hp.dev_bf16(qb), 1), padded(hp.dev_bf16(gb), 1)
    ks, vs = ([padded(hp.dev_bf16(x[i]), 1) for x in kv] for i in range(2))
    rows = [padded(torch.from_numpy(x).cuda(), 2) for x in (lse, D)]
    new = lambda n, heads: torch.full((B, n, heads, d), float("nan"), device="cuda")
    dq, dk, dv = new(sq, Hq), [new(sk, Hkv) for sk in sks], [new(sk, Hkv) for sk in sks]
    print(B, Hq, Hkv, sq, sks, causal, flush=True)
    lib.burst_attn_steps_bwd(shapes, masks, q, ks, vs, g, *rows, dq, dk, dv)
    torch.cuda.synchronize()
    assert hp.rel_err(dq.cpu().numpy(), sum(r[0] for r in refs)) <= hp.REL_TOL
    for i, r in enumerate(refs):
        assert hp.rel_err(dk[i].cpu().numpy(), r[1]) <= hp.REL_TOL
        assert hp.rel_err(dv[i].cpu().numpy(), r[2]) <= hp.REL_TOL
