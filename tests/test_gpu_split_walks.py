"""Launches of few query tiles, whose four waves deal the walk among themselves, and of many, which take the kernels of one walk a wave.

The inputs are one batch entry's; a launch of few tiles has that one, a launch of many the same entry again and again, so that both
ways run on the same small shapes: walks of no, one, three, four, five and more tiles for four waves, ragged last tiles, rows that see nothing,
several steps, a window, a block mask, a live running state."""
import numpy as np
import pytest

from oracle import burst_oracle as oc
from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu

FEW, MANY = 1, 640      # batch entries: MANY x 2 heads are beyond the rule of both directions, however few rows
CASES = [  # query rows, key rows of each step, causal, window, block mask
    (1, (1,), False, 0, False),
    (33, (64, 65), False, 0, False),
    (31, (191,), True, 0, False),
    (64, (257, 1, 129), True, 0, False),
    (70, (320,), True, 90, False),
    (100, (449, 64), True, 40, False),
    (129, (300,), False, 0, True),
    (129, (513,), True, 200, True),
]


def _inputs(case, d):
    sq, sks, causal, window, blocks = case
    Hq, Hkv = 2, 1
    rng = np.random.Generator(np.random.PCG64(wl.BASE_SEED + 91000 + sq + d))
    draw = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    q, g = draw(1, sq, Hq, d), draw(1, sq, Hq, d)
    kv = [(draw(1, sk, Hkv, d), draw(1, sk, Hkv, d)) for sk in sks]
    pattern = None
    if blocks:
        pattern = rng.integers(0, 2, (-(-sq // 256), -(-sks[0] // 128))).astype(np.uint8)
        pattern[0, 1] = 1
    return Hq, Hkv, rng, q, g, kv, pattern


def _mask(lib, case, sk, first_key, pattern):
    sq, _, causal, window, _ = case
    m = lib.burst_mask_t()
    m.mode = lib.BURST_MASK_CAUSAL if causal else lib.BURST_MASK_FULL
    m.q_nseg = m.k_nseg = m.pos_stride = 1
    m.q_seg_len, m.k_seg_len, m.window = sq, sk, window
    m.q_seg_pos[0], m.k_seg_pos[0] = 140, first_key
    vis = oc.visibility(140 + np.arange(sq), first_key + np.arange(sk), causal, window)
    if pattern is not None:
        import torch
        on_gpu = torch.from_numpy(pattern).cuda()
        lib.set_block_mask(m, on_gpu, 256, 128)
        m.keep = on_gpu
        vis = oc.apply_block_mask(vis, pattern, 256, 128)
    return m, vis


@pytest.mark.parametrize("batch", [FEW, MANY])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", CASES, ids=[str(c[:4]) for c in CASES])
def test_forward(lib, case, d, batch):
    import torch
    sq, sks = case[:2]
    Hq, Hkv, rng, qb, _, kv, pattern = _inputs(case, d)
    print(case, d, batch, flush=True)
    scale = d ** -0.5
    O = rng.standard_normal((1, sq, Hq, d)).astype(np.float32)
    lse = rng.uniform(-2.0, 6.0, (1, Hq, sq)).astype(np.float32)
    lse[rng.random(lse.shape) < 0.3] = -np.inf
    many = lambda x: x.repeat(batch, *[1] * (x.dim() - 1))
    o_acc, lse_acc = many(torch.from_numpy(O).cuda()), many(torch.from_numpy(lse).cuda())
    O[np.transpose(lse == -np.inf, (0, 2, 1))] = 0.0
    O, lse = O.astype(np.float64), lse.astype(np.float64)
    masks, ks, vs, at = [], [], [], 0
    for (kb, vb), sk in zip(kv, sks):
        m, vis = _mask(lib, case, sk, at, pattern)
        at += sk
        masks.append(m)
        ks.append(many(hp.dev_bf16(kb)))
        vs.append(many(hp.dev_bf16(vb)))
        if sk:
            part = oc.mha_step_fwd(hp.widen(qb), hp.widen(kb), hp.widen(vb), scale, vis)
            O, lse = oc.mha_lse_merge(O, lse, *part)
    q = many(hp.dev_bf16(qb))
    if len(sks) == 1:
        shp = lib.shape(batch, Hq, Hkv, d, sq, sks[0], scale)
        o_part, lse_part = torch.full_like(o_acc, 7.0), torch.full_like(lse_acc, 7.0)
        lib.burst_attn_step_fwd(shp, masks[0], q, ks[0], vs[0], o_part=o_part, lse_part=lse_part, o_acc=o_acc, lse_acc=lse_acc)
        torch.cuda.synchronize()
        got, got_lse = o_part.cpu().numpy(), lse_part.cpu().numpy()
        assert np.array_equal(got, np.broadcast_to(got[:1], got.shape)) and np.array_equal(got_lse, np.broadcast_to(got_lse[:1], got_lse.shape))
        assert hp.rel_err(got[:1], part[0]) <= hp.REL_TOL
        assert hp.lse_err(got_lse[:1], part[1]) <= hp.LSE_TOL
    else:
        shapes = [lib.shape(batch, Hq, Hkv, d, sq, sk, scale) for sk in sks]
        lib.burst_attn_steps_fwd(shapes, masks, q, ks, vs, o_acc, lse_acc)
        torch.cuda.synchronize()
    got, got_lse = o_acc.cpu().numpy(), lse_acc.cpu().numpy()
    live = np.broadcast_to(lse > -np.inf, got_lse.shape)      # (a row nothing was ever seen of keeps what it held)
    assert np.array_equal(got, np.broadcast_to(got[:1], got.shape))
    rows = np.transpose(live, (0, 2, 1))[:1]
    assert hp.rel_err(got[:1][rows], O[rows]) <= hp.REL_TOL
    assert hp.lse_err(got_lse[:1], lse) <= hp.LSE_TOL


@pytest.mark.parametrize("batch", [FEW, MANY])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", CASES, ids=[str(c[:4]) for c in CASES])
def test_backward(lib, case, d, batch):
    import torch
    sq, sks = case[:2]
    Hq, Hkv, rng, qb, gb, kv, pattern = _inputs(case, d)
    print(case, d, batch, flush=True)
    scale = d ** -0.5
    lse = rng.normal(4.0, 0.3, (1, Hq, sq)).astype(np.float32)
    lse[0, 0, sq // 2] = -np.inf      # a row that saw nothing in the whole ring
    D = rng.standard_normal((1, Hq, sq)).astype(np.float32)
    many = lambda x: x.repeat(batch, *[1] * (x.dim() - 1))
    masks, ks, vs, refs, at = [], [], [], [], 0
    for (kb, vb), sk in zip(kv, sks):
        m, vis = _mask(lib, case, sk, at, pattern)
        at += sk
        masks.append(m)
        ks.append(many(hp.dev_bf16(kb)))
        vs.append(many(hp.dev_bf16(vb)))
        seen = np.ones((sq, sk), bool) if vis is None else vis.copy()
        ref = [np.zeros((1, sq, Hq, d)), np.zeros((1, sk, Hkv, d)), np.zeros((1, sk, Hkv, d))]
        for h in range(Hq):               # head by head: the row without keys is one head's
            mine = seen.copy()
            mine[~np.isfinite(lse[0, h])] = False
            lse_h = np.where(np.isfinite(lse[:, h:h + 1]), lse[:, h:h + 1], 0.0).astype(np.float64)
            one = oc.mha_step_bwd(hp.widen(qb)[:, :, h:h + 1], hp.widen(kb), hp.widen(vb), hp.widen(gb)[:, :, h:h + 1], lse_h,
                                  D[:, h:h + 1].astype(np.float64), scale, mine)
            ref[0][:, :, h:h + 1] += one[0]
            ref[1] += one[1]
            ref[2] += one[2]
        refs.append(ref)
    prior = rng.standard_normal((1, sq, Hq, d)).astype(np.float32)
    dq = many(torch.from_numpy(prior).cuda())
    nan = lambda sk: torch.full((batch, sk, Hkv, d), float("nan"), device="cuda")
    dks, dvs = [nan(sk) for sk in sks], [nan(sk) for sk in sks]
    args = [many(hp.dev_bf16(gb)), many(torch.from_numpy(lse).cuda()), many(torch.from_numpy(D).cuda())]
    q = many(hp.dev_bf16(qb))
    shapes = [lib.shape(batch, Hq, Hkv, d, sq, sk, scale) for sk in sks]
    if len(sks) == 1:
        lib.burst_attn_step_bwd(shapes[0], masks[0], q, ks[0], vs[0], *args, dq=dq, dk=dks[0], dv=dvs[0], accumulate_flags=lib.BURST_ACC_DQ)
    else:
        lib.burst_attn_steps_bwd(shapes, masks, q, ks, vs, *args, dq, dks, dvs, accumulate_flags=lib.BURST_ACC_DQ)
    torch.cuda.synchronize()
    want = [("dQ", dq, prior + sum(r[0] for r in refs))]
    want += [(f"{n}{i}", t[i], r[m]) for i, r in enumerate(refs) for n, t, m in (("dK", dks, 1), ("dV", dvs, 2))]
    # one scale for all steps' gradients of a kind: a step of a single key has small ones
    top = {n: max(np.abs(x).max() for m, _, x in want if m[:2] == n) for n in ("dQ", "dK", "dV")}
    for name, t, ref in want:
        got = t.cpu().numpy()
        assert np.array_equal(got, np.broadcast_to(got[:1], got.shape)), name
        assert np.abs(got[:1] - ref).max() <= hp.REL_TOL * top[name[:2]], name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", CASES + [(96, (1500, 700), True, 0, False), (50, (1000,), False, 0, False)], ids=lambda c: str(c[:4]))
def test_forward_does_not_depend_on_the_batch(lib, case, d):
    """The same rows from a launch of few tiles and from one of many: P is rounded to bf16 against the same maximum either way, and what
    is left is the order of fp32 sums.  Up to 2200 keys, 35 tiles of 64: the products and rescalings of 35 tiles and four waves' sums,
    each 2^-24 of at most the largest |V|, 4: 1e-5 of it, where P against maxima that differ, 2^-9 a key, is 1e-3."""
    import torch
    sq, sks = case[:2]
    Hq, Hkv, _, qb, _, kv, pattern = _inputs(case, d)
    scale = d ** -0.5
    got = []
    for batch in (FEW, MANY):
        print(case, d, batch, flush=True)
        many = lambda x: x.expand(batch, *x.shape[1:])     # (inputs may share memory)
        masks, ks, vs, at = [], [], [], 0
        for (kb, vb), sk in zip(kv, sks):
            masks.append(_mask(lib, case, sk, at, pattern)[0])
            at += sk
            # keys that grow along the chunk: a maximum that rises from tile to tile
            k = hp.dev_bf16(kb) * (1 + torch.arange(sk, device="cuda") / sk)[:, None, None]
            ks.append(many(k.to(torch.bfloat16)))
            vs.append(many(hp.dev_bf16(vb)))
        q = many(hp.dev_bf16(qb))
        o = torch.zeros((batch, sq, Hq, d), device="cuda")
        lse = torch.full((batch, Hq, sq), -np.inf, device="cuda")
        out = [o, lse]
        if len(sks) == 1:
            part = [torch.full_like(o, 7.0), torch.full_like(lse, 7.0)]
            lib.burst_attn_step_fwd(lib.shape(batch, Hq, Hkv, d, sq, sks[0], scale), masks[0], q, ks[0], vs[0], o_part=part[0],
                                    lse_part=part[1], o_acc=o, lse_acc=lse)
            out += part
        else:
            lib.burst_attn_steps_fwd([lib.shape(batch, Hq, Hkv, d, sq, sk, scale) for sk in sks], masks, q, ks, vs, o, lse)
        torch.cuda.synchronize()
        got.append([x[:1].cpu().numpy() for x in out])
    for few, many in zip(*got):
        live = np.isfinite(many)
        assert np.array_equal(np.isfinite(few), live)
        assert np.abs(few[live] - many[live]).max(initial=0.0) <= 4e-5
