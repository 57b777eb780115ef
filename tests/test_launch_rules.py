"""Which kernels the launches of a call take (host rules, no GPU), held against the walks of every tile under the mask: the rules look
at a few tiles only.  Where the walks of a work-group are dealt to its waves is a matter of speed; the limits are those the rules state."""
import random

import pytest

from tests import helpers as hp

SLACK = 1.3          # a few tiles stand for all


def plan(lib, call, masks, batch, q_heads, kv_heads, d):
    shapes = [lib.shape(batch, q_heads, kv_heads, d, m.q_nseg * m.q_seg_len, m.k_nseg * m.k_seg_len, d ** -0.5) for m in masks]
    return lib.burst_attn_launch_plan(call, shapes, masks)


def walks(lib, mask, of_queries, rows=32):
    """Tiles of 64 rows of the other axis that the tiles of `rows` rows of one axis walk."""
    n = mask.q_nseg * mask.q_seg_len if of_queries else mask.k_nseg * mask.k_seg_len
    return [lib.burst_attn_visible_tile_runs(mask, not of_queries, 64, r0, min(r0 + rows, n))[0][1] for r0 in range(0, n, rows)]


def forward_load(lib, masks, heads, d):
    """Work-groups of 32 query rows, in units of one with the longest walk, and up to how many of them the walks are dealt."""
    w = [sum(x) for x in zip(*(walks(lib, m, True) for m in masks))]
    return heads * sum(w) / max(w) if max(w) else 0.0, 520 if d == 128 else 544 if max(w) < 64 else 800


@pytest.mark.parametrize("kind,G,dev,j,rows,window,N_blk", [
    ("zigzag", 8, 3, 4, 16384, 6000, 0),            # the shard one place ahead: only rows in the middle see its keys
    ("zigzag", 8, 3, 4, 65536, 6000, 0),
    ("zigzag", 8, 3, 4, 65536, 30000, 0),
    ("block_striped", 2, 0, 1, 16384, 400, 1024),   # a window shorter than a device's share of a block: the end of each piece sees none
    ("causal", 1, 0, 0, 16384, 1000, 0),            # all walks alike but the first few
])
@pytest.mark.parametrize("d", [64, 128])
def test_launches_of_many_tiles_under_a_window(lib, kind, G, dev, j, rows, window, N_blk, d):
    mask = hp.fill_mask(lib, kind, dev, j, G, rows * G, window, N_blk)
    load, limit = forward_load(lib, [mask], 32, d)
    assert load > 2 * limit
    for call in ("fwd", "fwd_part"):
        assert plan(lib, call, [mask], 1, 32, 32, d) == [0]


@pytest.mark.parametrize("kind,heads,rows,d,dealt", [
    ("full", 16, 1024, 128, True), ("full", 17, 1024, 128, False),      # 512 and 544 work-groups, all alike
    ("full", 17, 1024, 64, True), ("full", 18, 1024, 64, False),        # short walks
    ("full", 6, 4096, 64, True), ("full", 7, 4096, 64, False),          # 768 and 896, walks of 64 tiles
    ("causal", 8, 4096, 128, True), ("causal", 9, 4096, 128, False),    # 1024 and 1152 that walk half of the longest
    ("causal", 12, 4096, 64, True), ("causal", 13, 4096, 64, False),
])
def test_the_line_of_the_forward_rule(lib, kind, heads, rows, d, dealt):
    mask = hp.fill_mask(lib, kind, 0, 0, 1, rows)
    assert plan(lib, "fwd", [mask], 1, heads, heads, d) == [lib.BURST_KERNEL_DEALT if dealt else 0]


def test_few_tiles_are_dealt(lib):
    for kind, heads, rows in (("full", 2, 256), ("causal", 4, 1024), ("causal", 1, 16384), ("zigzag", 8, 1024)):
        assert plan(lib, "fwd", [hp.fill_mask(lib, kind, 0, 0, 1, rows)], 1, heads, heads, 128) == [lib.BURST_KERNEL_DEALT]
    both = lib.BURST_KERNEL_DQ | lib.BURST_KERNEL_DKDV
    assert plan(lib, "bwd", [hp.fill_mask(lib, "full", 0, 0, 1, 256)], 1, 2, 2, 128) == [both | lib.BURST_KERNEL_DEALT]
    assert plan(lib, "bwd", [hp.fill_mask(lib, "full", 0, 0, 1, 1024)], 1, 12, 12, 128) == [both | lib.BURST_KERNEL_KEY_TILES_64]


def backward_times(lib, masks, batch, q_heads, kv_heads, d):
    """The rule's two times, of dealt walks and of the other kernels, from all walks."""
    keys, group = batch * kv_heads, q_heads // kv_heads
    q = [sum(x) for x in zip(*(walks(lib, m, True) for m in masks))]
    k = [walks(lib, m, False) for m in masks]
    dq, dkdv = max(q), group * max(max(x) for x in k)
    work = keys * group * (3 * sum(q) + 4 * sum(sum(x) for x in k))
    groups = keys * group * sum(x > 0 for x in q) + keys * sum(x > 0 for w in k for x in w)
    return max(3 * dq, 4 * dkdv, work / 256) + (groups - 1) // 256 * 8, max((6 if d == 128 else 8) * dq, (3 if d == 128 else 4) * dkdv)


@pytest.mark.parametrize("seed", range(240))
def test_a_few_tiles_stand_for_all(lib, seed):
    rng = random.Random(seed)
    kind = rng.choice(["full", "causal", "zigzag", "striped", "block_striped"])
    G = rng.choice([1, 2, 4, 8])
    dev = rng.randrange(G)
    per = rng.choice([64, 256, 512])
    rows = per * rng.randint(2, 24) if kind == "block_striped" else 2 * rng.randint(30, 6000)
    window = 0 if kind == "full" or rng.random() < 0.4 else rng.randint(50, rows * G)
    masks = [hp.fill_mask(lib, kind, dev, (dev - t) % G, G, rows * G, window, per * G) for t in range(rng.randint(1, min(G, 4)))]
    batch, kv, group, d = rng.choice([1, 1, 2]), rng.choice([1, 2, 4, 8, 16]), rng.choice([1, 1, 4]), rng.choice([64, 128])
    if len(masks) == 1:
        f, limit = forward_load(lib, masks, batch * kv * group, d)
        got = plan(lib, "fwd", masks, batch, kv * group, kv, d)
        if f == 0:
            assert got == []
        elif not limit / SLACK < f < limit * SLACK:
            assert got == [lib.BURST_KERNEL_DEALT if f <= limit else 0], f
    masks = [m for m in masks if any(walks(lib, m, True))]
    got = plan(lib, "bwd", masks, batch, kv * group, kv, d) if masks else []
    if len(got) == 1 and got[0] & lib.BURST_KERNEL_DQ and got[0] & lib.BURST_KERNEL_DKDV:
        dealt, other = backward_times(lib, masks, batch, kv * group, kv, d)
        if not other / SLACK < dealt < other * SLACK:
            assert bool(got[0] & lib.BURST_KERNEL_DEALT) == (dealt <= other), (dealt, other)


def test_launch_plan_refuses_what_the_calls_refuse(lib):
    mask = hp.fill_mask(lib, "causal", 0, 0, 1, 512)
    other = hp.fill_mask(lib, "causal", 0, 0, 1, 256)
    for call, masks, heads in (("fwd_part", [mask, mask], 2), ("fwd", [mask, other], 2), ("fwd", [mask], 3)):
        with pytest.raises(lib.BurstError):
            plan(lib, call, masks, 1, heads, 2, 128)
    assert plan(lib, "fwd", [mask, mask], 1, 2, 2, 128) == [lib.BURST_KERNEL_DEALT]


@pytest.mark.parametrize("N,d,v,tile,edges", [
    (207, 2560, 10874, 256, [128, 128, 256]), (2426, 768, 8354, 4096, [128, 256, 128]),
    (1000, 256, 15361, 1024, [256, 128, 128]), (16384, 4096, 32000, 8192, [256, 256, 256]),
])
def test_tiles_of_the_lm_head(lib, N, d, v, tile, edges):
    assert [edge for edge, _ in lib.burst_lm_head_tile_plan(lib.lm_head_shape(N, d, v, tile))] == edges


def test_tile_plan_of_the_lm_head_refuses_what_the_call_refuses(lib):
    for shape in ((0, 256, 64, 256), (64, 200, 64, 256), (64, 256, 64, 200)):
        with pytest.raises(lib.BurstError):
            lib.burst_lm_head_tile_plan(lib.lm_head_shape(*shape))
