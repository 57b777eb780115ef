"""Host run of the decisions a wave takes in its walk (class of a tile, rows a lane's row sees) against brute force over
positions: what the kernels compile, compiled for the CPU."""
import ctypes as C
import glob
import os
import re

import numpy as np
import pytest

from oracle import burst_oracle as oc
from tests import helpers as hp

LAST = 2 ** 31 - 1   # the position behind the last row stays below it


def _mask(lib, q_pos, k_pos, q_len, k_len, q_nseg=1, k_nseg=1, stride=1, window=0, causal=True):
    m = lib.burst_mask_t()
    m.mode = lib.BURST_MASK_CAUSAL if causal else lib.BURST_MASK_FULL
    m.q_nseg, m.k_nseg, m.q_seg_len, m.k_seg_len, m.pos_stride, m.window = q_nseg, k_nseg, q_len, k_len, stride, window
    for s, p in enumerate(q_pos):
        m.q_seg_pos[s] = p
    for s, p in enumerate(k_pos):
        m.k_seg_pos[s] = p
    return m


def _masks(lib):
    for window in (0, 1, 50, 333, 5000, LAST - 1):
        yield _mask(lib, (100,), (0,), 300, 400, window=window)
        yield _mask(lib, (0,), (900,), 300, 100, window=window)                          # every key behind every query
        yield _mask(lib, (90, 700), (0, 350), 150, 170, 2, 2, window=window)             # two pieces: the path without divisions
        yield _mask(lib, (90, 700), (200,), 150, 333, 2, 1, window=window)
        yield _mask(lib, (500,), (0, 350), 333, 70, 1, 2, window=window)
        yield _mask(lib, (40,), (7,), 333, 200, stride=3, window=window)
        yield _mask(lib, (7, 507), (0, 650), 100, 150, 2, 2, stride=3, window=window)    # two pieces with a stride
        yield _mask(lib, (7, 307), (0, 450), 100, 150, 5, 3, stride=2, window=window)
        yield _mask(lib, (0, 96), (32, 128), 32, 32, 7, 7, window=window)
        yield _mask(lib, (LAST - 300,), (LAST - 500,), 300, 400, window=window)          # the last positions there are
        yield _mask(lib, (LAST - 1000, LAST - 300), (3, LAST - 200), 300, 200, 2, 2, window=window)
        yield _mask(lib, (LAST - 5 * 1000, LAST - 4 * 1000), (0, LAST // 4), 100, 150, 5, 4, window=window)
        yield _mask(lib, (LAST - 100 * 1000,), (5,), 100, 300, stride=1000, window=window)
    yield _mask(lib, (0,), (0,), 130, 70, causal=False)
    yield _mask(lib, (0, 512), (0, 512), 100, 130, 2, 2, causal=False)


def _vis(lib, m):
    return oc.visibility(hp.mask_positions(m, "q"), hp.mask_positions(m, "k"), m.mode == lib.BURST_MASK_CAUSAL, m.window)


def test_rows_that_a_row_sees_match_brute_force(lib):
    for n, m in enumerate(_masks(lib)):
        vis = _vis(lib, m)
        for query_axis, seen in ((0, vis), (1, vis.T)):
            for row in range(seen.shape[0]):
                lo, hi = lib.burst_attn_visible_rows(m, query_axis, row)
                want = np.flatnonzero(seen[row])
                if want.size == 0:
                    assert lo >= hi, (n, query_axis, row, lo, hi)
                else:
                    assert (lo, hi) == (want[0], want[-1] + 1) and want.size == hi - lo, (n, query_axis, row, lo, hi)


def test_tile_classes_of_a_walk_match_brute_force(lib):
    """Tiles of a walk (heights of the kernels: 64, and 32 query rows where two wave pairs share 32 keys) against 32 own
    rows.  A verdict of "nothing" or "all" is what counts: it must be right wherever it is given, and without a window it
    is given wherever it is right."""
    for n, m in enumerate(_masks(lib)):
        vis = _vis(lib, m)
        sq, sk = vis.shape
        for method, hq, hk in ((1, 64, 32), (1, 32, 32), (2, 32, 64), (3, 64, 32), (4, 32, 64)):
            for q0 in range(0, sq, hq):
                for k0 in range(0, sk, hk):
                    q1, k1 = min(q0 + hq, sq), min(k0 + hk, sk)
                    sub = vis[q0:q1, k0:k1]
                    whole = method < 3 or (q0 + 64 <= sq if method == 3 else k0 + 64 <= sk)
                    want = 0 if not sub.any() else 1 if sub.all() and whole else 2
                    got = lib.burst_attn_tile_class(m, q0, q1, k0, k1, method)
                    assert got == want or (m.window and got == 2), (n, method, q0, k0, got, want)


@pytest.mark.parametrize("row", [-1, 300])
def test_visible_rows_rejects_bad_arguments(lib, row):
    raw, out = lib.raw(), (C.c_int32 * 2)()
    m = _mask(lib, (100,), (0,), 300, 400)
    assert raw.burst_attn_visible_rows(C.byref(m), 0, row, C.byref(out)) == lib.BURST_ERR_INVALID_ARG
    assert raw.burst_attn_visible_rows(None, 0, 0, C.byref(out)) == lib.BURST_ERR_INVALID_ARG
    assert raw.burst_attn_visible_rows(C.byref(m), 0, 0, None) == lib.BURST_ERR_INVALID_ARG


def test_no_build_flag_sets_the_rows_of_a_work_group():
    """Plans, grids and kernels of a launch, and the two kernels of a joint launch, share one constant."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_19836_amd", "csrc")
    flags = {name for path in glob.glob(os.path.join(csrc, "*")) for name in re.findall(r"#ifndef (BURST_\w+)", open(path).read())}
    assert flags == {"BURST_MFMA_PRIO", "BURST_A16"}   # wave priority of MFMA streams, operands fetched ahead
