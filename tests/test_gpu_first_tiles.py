"""The first two key tiles of a walk, with key rows so far apart that the loads of each tile take long.

Eight waves bring a tile together, and the waves of one half start on a tile a phase before those of the other: each
must find the other half's share of the second tile there as well.  That is so where the kernels of one walk a wave run: the
launches here have few tiles and deal their walks, each wave with tiles of its own; test_gpu_whole_walks.py runs the same on the others."""
import numpy as np
import pytest

from oracle import burst_oracle as oc
from paper_2509_19836_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu

ROW_STRIDE = 1 << 19   # elements between key rows: a page each


@pytest.mark.parametrize("sk", [64, 65, 128, 190, 300])
@pytest.mark.parametrize("d", [64, 128])
def test_first_key_tiles_with_scattered_rows(lib, d, sk):
    import torch
    B, Hq, Hkv, sq = 1, 8, 8, 256
    rng = np.random.Generator(np.random.PCG64(wl.BASE_SEED + 72000 + d + sk))
    draw = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    qb, kb, vb = draw(B, sq, Hq, d), draw(B, sk, Hkv, d), draw(B, sk, Hkv, d)
    O_ref, lse_ref = oc.mha_step_fwd(hp.widen(qb), hp.widen(kb), hp.widen(vb), d ** -0.5, None)
    q, k, v = hp.dev_bf16(qb), hp.dev_bf16(kb), hp.dev_bf16(vb)
    scattered = lambda x: (lambda t: (t.copy_(x), t)[1])(torch.empty(sk * ROW_STRIDE, device="cuda", dtype=torch.bfloat16)
                                                         .as_strided((B, sk, Hkv, d), (0, ROW_STRIDE, d, 1)))
    k, v = scattered(k), scattered(v)
    shp = lib.shape(B, Hq, Hkv, d, sq, sk, d ** -0.5)
    first = None
    for _ in range(4):   # nothing but rounding separates the result from the oracle's, and nothing two passes
        o = torch.empty((B, sq, Hq, d), device="cuda", dtype=torch.float32)
        lse = torch.empty((B, Hq, sq), device="cuda", dtype=torch.float32)
        lib.burst_attn_step_fwd(shp, None, q, k, v, o_part=o, lse_part=lse)
        torch.cuda.synchronize()
        got = o.cpu().numpy(), lse.cpu().numpy()
        assert hp.rel_err(got[0], O_ref) <= hp.REL_TOL
        assert hp.lse_err(got[1], lse_ref) <= hp.LSE_TOL
        if first is not None:
            assert np.array_equal(got[0], first[0]) and np.array_equal(got[1], first[1])
        first = got
