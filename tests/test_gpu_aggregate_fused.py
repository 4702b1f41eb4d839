"""The fused aggregation at the edges of its tiles and steps: every degree, one
and several column groups (the last one partly empty), heads narrower and wider
than a group, rows of 0, 1, 16, 17 and more edges, with and without weights,
both filters, against the oracle's layer.  Run with -m gpu."""
import numpy as np
import pytest
import torch

import e2f_synth as syn
import oracle as o
from cases import TOL_F32

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def gpu(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# float products and sums of at most 49 x 64 terms a value, coupled once: the
# parity bar 1e-4 of the layer leaves two digits over the 1e-6 seen
@pytest.mark.parametrize("L,C,H", [(0, 4, 1), (1, 12, 3), (2, 36, 3), (2, 16, 4), (3, 32, 8), (3, 100, 5), (4, 4, 1),
                                   (4, 48, 4), (4, 64, 1), (5, 4, 1), (5, 40, 2), (5, 64, 8), (6, 4, 1), (6, 48, 4),
                                   (6, 32, 1), (0, 20, 1), (1, 24, 2), (2, 20, 5), (2, 64, 4), (1, 144, 9), (5, 20, 1),
                                   (5, 144, 3)])
@pytest.mark.parametrize("y_norm", [False, True])
def test_tile_edges(L, C, H, y_norm):
    import paper_2501_19216_amd as e2f
    ctx = e2f.e2f_create(L, 0)
    try:
        rng = np.random.default_rng(7 * L + C)
        n = 41
        pos = syn.quantize(rng.uniform(0, 6.0, size=(n, 3)))
        # row i: its length cycles through the edges of a step of 16
        deg = [(0, 1, 4, 5, 15, 16, 17, 32, 33, 40)[i % 10] for i in range(n)]
        rows = [np.sort(rng.choice(np.delete(np.arange(n), i), size=d, replace=False)) for i, d in enumerate(deg)]
        rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
        ci = np.concatenate(rows).astype(np.int32)
        feat = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
        alpha = rng.uniform(0.1, 1.0, size=(len(ci), H)).astype(np.float32)
        w = rng.uniform(0.5, 1.5, size=(L + 1) ** 3)
        ref = o.layer(L, H, pos, feat, rp, ci, alpha, w, y_norm=y_norm)
        one = o.layer(L, H, pos, feat, rp, ci, np.ones_like(alpha), w, y_norm=y_norm)
        print("L %d C %d H %d y_norm %s" % (L, C, H, y_norm), flush=True)
        for al, want in ((alpha, ref), (None, one)):
            got = e2f.e2f_wigner6j_conv_forward(ctx, gpu(pos), gpu(feat), gpu(rp), gpu(ci), gpu(al), L, H, 6.0, path_w=w,
                                                y_norm=y_norm).cpu().numpy()
            err = o.max_rel_err(got, want, L)
            print("  err %.3e" % err)
            assert err <= TOL_F32
            assert np.all(got[np.array(deg) == 0] == 0)
    finally:
        ctx.close()
