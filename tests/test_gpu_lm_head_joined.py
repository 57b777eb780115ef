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
    assert np.array_equal(loss, loss0) and np.array_equal(lse, lse0)      # (d < 2048: the logits are not split)
    norm = np.linalg.norm
    assert norm(d_w - d_w0) <= 1e-5 * norm(d_w0)                          # fp32 sums in another order
    # dH: the contraction may be split otherwise; in bf16 a sum that lies between two numbers may go to the other one
    assert norm(d_h - d_h0) <= (1e-5 if dh == "f32" else 1e-3) * norm(d_h0)
    assert np.abs(d_h - d_h0).max() <= (1e-5 if dh == "f32" else 2 ** -7) * np.abs(d_h0).max()
    if tile >= 512:
        assert np.array_equal(d_w, d_w0) and np.array_equal(d_h, d_h0)


@pytest.mark.parametrize("N,d,v,tile,parts", [(1, 2048, 300, 512, 2), (256, 3072, 2000, 1024, 3), (257, 2048, 1300, 1024, 2), (70, 4096, 900, 1024, 4)])
@pytest.mark.parametrize("grads", [True, False])
def test_logits_in_parts_equal_the_whole(lib, N, d, v, tile, parts, grads):
    """The contraction of the logits dealt to several work-groups (few output tiles, room in the buffer, 16 k-tiles of 64 a part)
    against a tile whose buffer has no room for that."""
    import torch
    Hb, Wb, Y = wl.lm_head_tensors(wl.BASE_SEED + 32000 + N, N, d, v, ignored=1 if N > 1 else 0)
    h, w, y = hp.dev_bf16(Hb), hp.dev_bf16(Wb), torch.from_numpy(Y).cuda()
    whole = -(-N // 256) * 256
    assert min(tile // whole, d // 1024) == parts
    out = []
    for B_s in (whole, tile):
        shp = lib.lm_head_shape(N, d, v, B_s, 1.0 / N)
        loss, lse = torch.full((N,), 7.0, device="cuda"), torch.full((N,), 7.0, device="cuda")
        d_h, d_w = torch.full((N, d), 7.0, device="cuda"), torch.full((v, d), 7.0, device="cuda")
        ws = torch.full((lib.burst_lm_head_workspace_bytes(shp),), 255, dtype=torch.uint8, device="cuda")
        print(f"lm head: N={N} d={d} v={v} tile={B_s}", flush=True)
        lib.burst_lm_head_loss(shp, h, w, y, loss, ws, lse=lse, d_h=d_h if grads else None, d_w=d_w if grads else None)
        torch.cuda.synchronize()
        out.append([t.double().cpu().numpy() for t in (loss, lse, d_h, d_w)])
    ref = (hp.widen(Hb) @ hp.widen(Wb).T)
    top = ref.max(1)
    lse_ref = top + np.log(np.exp(ref - top[:, None]).sum(1))
    for loss, lse, _, _ in out:
        # fp32 sums of d products of size about |logit| / sqrt(d): 1e-6 of the largest logit, with room
        assert np.abs(lse - lse_ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())
    (loss0, lse0, dh0, dw0), (loss1, lse1, dh1, dw1) = out
    assert np.abs(loss0 - loss1).max() <= 2e-5 * max(1.0, np.abs(ref).max())
    norm = np.linalg.norm
    # dLogits is bf16: a sum that lies between two numbers may go to the other one
    assert norm(dh1 - dh0) <= 1e-3 * norm(dh0) and norm(dw1 - dw0) <= 1e-3 * norm(dw0)
