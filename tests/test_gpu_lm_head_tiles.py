"""The LM head's GEMM loop at the edges of its tiles: one to five k-tiles in each of the three products, a last k-tile
of one to 64 words, a last token or word tile of one row, matrices that end where memory full of NaN begins."""
import numpy as np
import pytest

from oracle import lm_head_oracle as lm
from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N, d, v, B_s, dh_dtype", [
    (1, 256, 63, 256, "f32"),      # one k-tile of 63 words; one k-tile of one token
    (64, 256, 64, 256, "bf16"),    # exactly one k-tile
    (65, 512, 65, 256, "f32"),     # two k-tiles, the second of one word / one token
    (193, 256, 257, 256, "f32"),   # a word tile of one row; five k-tiles, the last of one word
    (257, 512, 320, 512, "bf16"),  # a token tile of one row; five whole k-tiles
    (513, 768, 190, 256, "f32"),   # three sequence tiles, the last of one token; three k-tiles
    (300, 256, 5000, 256, "bf16"), # the vocabulary in many k-tiles
])
def test_edges(lib, N, d, v, B_s, dh_dtype):
    import torch
    Hb, Wb, Y = wl.lm_head_tensors(wl.BASE_SEED + 21000 + v, N, d, v, min(1, N - 1))
    gs = 1.0 / N
    loss_ref, lse_ref, dH_ref, dW_ref = lm.lm_head_loss(hp.widen(Hb), hp.widen(Wb), Y, gs)
    shp = lib.lm_head_shape(N, d, v, B_s, gs)
    nan = dict(device="cuda", fill_value=float("nan"))
    ws = torch.full((lib.burst_lm_head_workspace_bytes(shp),), 0xFF, dtype=torch.uint8, device="cuda")
    h, w = (torch.full((rows + 300, d), dtype=torch.bfloat16, **nan) for rows in (N, v))
    h[:N], w[:v] = hp.dev_bf16(Hb), hp.dev_bf16(Wb)
    loss, lse = (torch.full((N + 300,), dtype=torch.float32, **nan) for _ in range(2))
    dh = torch.full((N + 300, d), dtype=torch.float32 if dh_dtype == "f32" else torch.bfloat16, **nan)
    dw = torch.full((v + 300, d), dtype=torch.float32, **nan)
    print(f"lm head edges N={N} d={d} v={v} B_s={B_s} dh={dh_dtype}", flush=True)
    lib.burst_lm_head_loss(shp, h[:N], w[:v], torch.from_numpy(Y).cuda(), loss[:N], ws, lse=lse[:N], d_h=dh[:N], d_w=dw[:v])
    torch.cuda.synchronize()
    for got, ref, rows in ((loss, loss_ref, N), (lse, lse_ref, N), (dh, dH_ref, N), (dw, dW_ref, v)):
        assert torch.isnan(got[rows:]).all()       # nothing is written past the end
        got = got[:rows].float().cpu().numpy()
        tol = hp.LSE_TOL if got.ndim == 1 else hp.REL_TOL * max(np.abs(ref).max(), 1e-30)
        assert np.abs(got - ref).max() <= tol      # (false for NaN)
