"""Words whose logits are -inf (a vocabulary padded or masked by a bias column, or products past the fp32 range), NaN words: with
the logits contracted whole and in parts.

The masked words are groups of 8, 128 and 256 at positions that the parts' loss kernel (8 words a thread, 8192 a pass) meets first,
later and last, and one word alone."""
import numpy as np
import pytest
import torch

from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu

N, D, V = 64, 2048, 20000
CLOSED = np.r_[0:8, 5000, 8192:8200, 12032:12160, 16384:16640, V - 8:V]
TILES = {"whole": 256, "parts": 1024}   # the buffer of a tile of 256 has no room for parts


def _run(lib, h, w, y, tile):
    shp = lib.lm_head_shape(N, D, V, tile, 1.0 / N)
    loss, lse = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
    d_h, d_w = torch.empty(N, D, device="cuda"), torch.empty(V, D, device="cuda")
    ws = torch.full((lib.burst_lm_head_workspace_bytes(shp),), 255, dtype=torch.uint8, device="cuda")
    print(f"lm head: N={N} d={D} v={V} tile={tile}", flush=True)
    lib.burst_lm_head_loss(shp, h, w, y, loss, ws, lse=lse, d_h=d_h, d_w=d_w)
    torch.cuda.synchronize()
    return [t.double().cpu().numpy() for t in (loss, lse, d_h, d_w)]


def _inputs(hidden, weight, closed):
    Hb, Wb, Y = wl.lm_head_tensors(wl.BASE_SEED + 33000, N, D, V, ignored=1)
    h, w = (torch.from_numpy(hp.widen(x)).to(torch.bfloat16) for x in (Hb, Wb))
    h[:, 0], w[:, 0] = hidden, 0.0
    w[torch.from_numpy(closed), 0] = weight
    Y = np.where((Y >= 0) & np.isin(Y, closed), 9, Y)
    return h, w, Y


@pytest.mark.parametrize("how", TILES)
@pytest.mark.parametrize("hidden, weight", [(1.0, -np.inf), (2.0 ** 64, -2.0 ** 66)], ids=["bias of -inf", "overflow"])
def test_words_at_minus_infinity_have_no_share(lib, how, hidden, weight):
    h, w, Y = _inputs(hidden, weight, CLOSED)
    loss, lse, d_h, d_w = _run(lib, h.cuda(), w.cuda(), torch.from_numpy(Y).cuda(), TILES[how])
    H, W = h.double().numpy(), w.double().numpy()
    open_words = np.setdiff1d(np.arange(V), CLOSED)
    x = H[:, 1:] @ W[open_words, 1:].T                 # (column 0 of the open words is zero)
    top = x.max(1)
    ref = top + np.log(np.exp(x - top[:, None]).sum(1))
    kept = (Y >= 0) & (Y < V)
    at = np.searchsorted(open_words, Y[kept])
    # fp32 sums of 2048 products: 1e-6 of the largest logit, with room
    bound = 1e-5 * max(1.0, np.abs(x).max())
    assert np.abs(lse - ref).max() <= bound
    assert np.abs(loss[kept] - (ref[kept] - x[kept, at])).max() <= bound
    dl = np.exp(x - ref[:, None])
    dl[np.flatnonzero(kept), at] -= 1.0
    dl[~kept] = 0.0
    dl /= N
    assert not d_w[CLOSED].any()
    for cols in (slice(0, 1), slice(1, D)):            # dLogits is bf16: 2^-9 a value
        assert hp.rel_err(d_w[open_words][:, cols], dl.T @ H[:, cols]) <= hp.REL_TOL
    assert hp.rel_err(d_h[:, 1:], dl @ W[open_words, 1:]) <= hp.REL_TOL
    if np.isfinite(weight):                            # (0 * -inf is NaN in the column of the bias)
        assert not d_h[:, 0].any()


@pytest.mark.parametrize("how", TILES)
@pytest.mark.parametrize("closed", [np.r_[8192:8200], np.r_[5000]], ids=["a group", "a word"])
def test_nan_words_reach_the_loss(lib, how, closed):
    h, w, Y = _inputs(1.0, np.nan, closed)
    loss, lse, _, _ = _run(lib, h.cuda(), w.cuda(), torch.from_numpy(Y).cuda(), TILES[how])
    assert np.isnan(lse).all() and np.isnan(loss[(Y >= 0) & (Y < V)]).all()
