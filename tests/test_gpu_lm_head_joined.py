"""Short sequence tiles of the call without a workspace, which the library joins: one tile and a row, one joined tile with a
ragged end, two of them (the array holds 1024 tokens at 40000 words), and tiles that are not joined."""
import numpy as np
import pytest

from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,v,tile", [(257, 512, 3000, 256), (700, 256, 900, 256), (1300, 256, 40000, 256), (256, 512, 2000, 256),
                                        (1100, 256, 5000, 512)])
@pytest.mark.parametrize("dh", ["bf16", "f32"])
def test_joined_tiles_equal_the_tiles_one_by_one(lib, N, d, v, tile, dh):
    import torch
    Hb, Wb, Y = wl.lm_head_tensors(wl.BASE_SEED + 31000 + N, N, d, v, ignored=3)
    h, w, y = hp.dev_bf16(Hb), hp.dev_bf16(Wb), torch.from_numpy(Y).cuda()
    shp = lib.lm_head_shape(N, d, v, tile, 1.0 / N)
    dt = torch.bfloat16 if dh == "bf16" else torch.float32
    out = {}
    for name in ("workspace", "noalloc"):
        print(f"lm head {name}: N={N} d={d} v={v} tile={tile}", flush=True)
        loss, lse = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
        d_h, d_w = torch.empty(N, d, device="cuda", dtype=dt), torch.full((v, d), 0.5, device="cuda")
        for accumulate in (False, True):     # the second call adds to the first one's dW
            kw = dict(lse=lse, d_h=d_h, d_w=d_w, accumulate_dw=accumulate)
            if name == "workspace":
                ws = torch.empty(lib.burst_lm_head_workspace_bytes(shp), dtype=torch.uint8, device="cuda")
                lib.burst_lm_head_loss(shp, h, w, y, loss, ws, **kw)
            else:
                lib.burst_lm_head_loss_noalloc(shp, h, w, y, loss, **kw)
        torch.cuda.synchronize()
        out[name] = [t.double().cpu().numpy() for t in (loss, lse, d_h, d_w)]
    (loss, lse, d_h, d_w), (loss0, lse0, d_h0, d_w0) = out["noalloc"], out["workspace"]
    assert np.array_equal(loss, loss0) and np.array_equal(lse, lse0)      # a token's logits do not depend on the tile
    norm = np.linalg.norm
    assert norm(d_w - d_w0) <= 1e-5 * norm(d_w0)                          # fp32 sums in another order
    # dH: the contraction may be split otherwise; in bf16 a sum that lies between two numbers may go to the other one
    assert norm(d_h - d_h0) <= (1e-5 if dh == "f32" else 1e-3) * norm(d_h0)
    assert np.abs(d_h - d_h0).max() <= (1e-5 if dh == "f32" else 2 ** -7) * np.abs(d_h0).max()
    if tile >= 512:
        assert np.array_equal(d_w, d_w0) and np.array_equal(d_h, d_h0)
