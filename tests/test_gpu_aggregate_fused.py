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


# Several receivers a workgroup, one after another (2 to 8, 64 apart in the
# order): the steps loaded ahead across rows, runs of empty rows between live
# ones, a last set that is not full, the partial sums of one receiver over those
# of the one before; receivers in their own order and sorted (above 8,192 atoms,
# and below where 3 GB of features are gathered: the last case).  Sampled rows
# against the oracle, every row against the two-kernel form, which shares neither
# kernel nor work split, every empty row zero.
@pytest.mark.parametrize("L,C,H,n", [(0, 128, 8, 20011), (1, 64, 4, 17003), (2, 128, 8, 5003), (2, 128, 4, 16403),
                                     (2, 48, 4, 7001), (3, 128, 8, 2501), (3, 64, 8, 9001), (4, 64, 4, 4099),
                                     (5, 64, 8, 1501), (5, 64, 4, 5003), (5, 48, 12, 1801), (6, 64, 8, 1301),
                                     (3, 1024, 8, 4003)])
def test_receivers_in_turn(L, C, H, n):
    import paper_2501_19216_amd as e2f
    ctx = e2f.e2f_create(L, 0)
    try:
        rng = np.random.default_rng(11 * L + C)
        pos = syn.quantize(rng.uniform(0, 6.0, size=(n, 3)))
        deg = np.array([(0, 0, 1, 16, 17, 0, 4, 33, 5, 15, 32, 0, 0, 40, 64)[i % 15] for i in range(n)])
        deg[n // 3:n // 3 + 400] = 0  # a run over several sets
        deg[-3:] = (0, 17, 0)
        rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
        ci = np.concatenate([np.sort(rng.choice(n - 1, size=d, replace=False)) for d in deg if d]).astype(np.int32)
        ci += ci >= np.repeat(np.arange(n), deg)  # (no atom is its own neighbour)
        feat = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
        alpha = rng.uniform(0.1, 1.0, size=(len(ci), H)).astype(np.float32)
        w = rng.uniform(0.5, 1.5, size=(L + 1) ** 3)
        print("L %d C %d H %d n %d" % (L, C, H, n), flush=True)
        args = (ctx, gpu(pos), gpu(feat), gpu(rp), gpu(ci), gpu(alpha), L, H, 6.0)
        got = e2f.e2f_wigner6j_conv_forward(*args, path_w=w).cpu().numpy()
        assert np.all(got[deg == 0] == 0)
        live = np.flatnonzero(deg)
        r = np.unique(np.concatenate([live[:16], live[-16:], rng.choice(live, size=32)])).astype(np.int32)
        ref = o.layer(L, H, pos, feat, rp, ci, alpha, w, rows=r)
        err = o.max_rel_err(got[r], ref, L)
        two = e2f.e2f_wigner6j_conv_forward(*args, path_w=w, form="split").cpu().numpy()
        every = o.max_rel_err(got, two, L)
        print("  err %.3e, against the two-kernel form %.3e" % (err, every))
        assert err <= TOL_F32 and every <= TOL_F32
    finally:
        ctx.close()


# Features of more than 2^32 bytes (64-bit offsets): senders on both sides of it.
@pytest.mark.parametrize("L,C,H", [(2, 1024, 8), (3, 1024, 16), (5, 1024, 4), (6, 1024, 8)])
def test_features_beyond_4_gib(L, C, H):
    import paper_2501_19216_amd as e2f
    nk = (L + 1) ** 2
    n = int(4.5e9 / (4 * nk * C))
    ctx = e2f.e2f_create(L, 0)
    try:
        rng = np.random.default_rng(5 + L)
        far = int(2 ** 32 / (4 * nk * C)) + 1  # the first atom past 2^32 bytes
        recv = np.sort(np.concatenate([[0, 1, far - 1, far, n - 1], rng.choice(np.arange(2, far - 1), 40, replace=False)]))
        deg = np.zeros(n, dtype=np.int64)
        deg[recv] = rng.integers(1, 40, size=len(recv))
        rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
        cols = [np.sort(np.concatenate([rng.choice(np.arange(far, n - 1), (d + 1) // 2, replace=False),
                                        rng.choice(np.arange(2, far - 1), d // 2, replace=False)])) for d in deg[recv]]
        ci = np.concatenate(cols).astype(np.int32)
        pos = syn.quantize(rng.uniform(0, 6.0, size=(n, 3)))
        g = torch.Generator(device=DEV).manual_seed(L)
        feat = torch.randn(n, nk, C, device=DEV, generator=g)
        alpha = rng.uniform(0.1, 1.0, size=(len(ci), H)).astype(np.float32)
        w = rng.uniform(0.5, 1.5, size=(L + 1) ** 3)
        print("L %d C %d H %d n %d: %.2f GB of features" % (L, C, H, n, feat.numel() * 4e-9), flush=True)
        size = e2f.e2f_wigner6j_workspace_size(ctx, n, len(ci), L, C, H, 6.0, path_w=w, minimum=True)
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        got = e2f.e2f_wigner6j_conv_forward(ctx, gpu(pos), feat, gpu(rp), gpu(ci), gpu(alpha), L, H, 6.0, path_w=w,
                                            workspace=ws)
        empty = torch.from_numpy(deg == 0).to(DEV)
        assert not bool((got.abs().amax(dim=(1, 2))[empty] != 0).any())
        # the graph of the atoms that take part, for the oracle
        used = np.unique(np.concatenate([recv, ci]))
        at = np.searchsorted(used, recv).astype(np.int32)
        ld = np.zeros(len(used), dtype=np.int64)
        ld[at] = deg[recv]
        lrp = np.concatenate([[0], np.cumsum(ld)]).astype(np.int64)
        sub = feat[torch.from_numpy(used).to(DEV)].cpu().numpy()
        ref = o.layer(L, H, pos[used], sub, lrp, np.searchsorted(used, ci).astype(np.int32), alpha, w, rows=at)
        err = o.max_rel_err(got[torch.from_numpy(recv).to(DEV)].cpu().numpy(), ref, L)
        print("  err %.3e" % err)
        assert err <= TOL_F32
    finally:
        ctx.close()
        torch.cuda.empty_cache()


@pytest.mark.parametrize("L,C,H,n", [(2, 64, 4, 900), (5, 128, 8, 300)])
def test_bf16_mixing_is_of_the_rounded_sums(L, C, H, n):
    # bf16 mixing rounds y to bf16 once: the mixed output equals the product of the
    # rounded unmixed output (float sums of C products: 1e-6 a product), so that two
    # correct y differ in it only where one lies near a tie
    import paper_2501_19216_amd as e2f
    ctx = e2f.e2f_create(L, 0)
    try:
        g = torch.Generator(device=DEV).manual_seed(3)
        pos = gpu(syn.quantize(np.random.default_rng(3).uniform(0, 14.0, size=(n, 3))))
        rp, ci = e2f.e2f_neighbor_list(ctx, pos, 6.0)
        feat = torch.randn(n, (L + 1) ** 2, C, device=DEV, generator=g)
        alpha = torch.rand(ci.numel(), H, device=DEV, generator=g)
        W = (torch.randn(L + 1, C, C, device=DEV, generator=g) / C ** 0.5).bfloat16()
        y = e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, 6.0)
        got = e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, 6.0, mix_w=W)
        for l in range(L + 1):
            a = y[:, l * l:(l + 1) ** 2].bfloat16().double().reshape(-1, C)
            ref = a @ W[l].double().t().contiguous()
            err = float((got[:, l * l:(l + 1) ** 2].double().reshape(-1, C) - ref).abs().max() / ref.abs().max())
            print("bf16 mixing L %d degree %d: %.3e" % (L, l, err), flush=True)
            assert err <= 4e-6
    finally:
        ctx.close()


@pytest.mark.parametrize("L,bad", [(2, np.inf), (4, np.inf), (4, np.nan), (6, -np.inf)])
def test_bad_values_stay_where_they_belong(L, bad):
    # a feature, weight or gradient that is not finite reaches the receivers (rows,
    # edges) that read it and no other value, which stays what it was bit for bit
    # (past a row's end its last sender is read with a weight of zero; receivers of
    # one workgroup follow each other in the same registers)
    import paper_2501_19216_amd as e2f
    C, H, n, j0, c0 = 32, 4, 700, 123, 7
    ctx = e2f.e2f_create(L, 0)
    try:
        g = torch.Generator(device=DEV).manual_seed(L)
        pos = gpu(syn.quantize(np.random.default_rng(L).uniform(0, 19.0, size=(n, 3))))
        rp, ci = e2f.e2f_neighbor_list(ctx, pos, 5.0)
        feat, gout = (torch.randn(n, (L + 1) ** 2, C, device=DEV, generator=g) for _ in range(2))
        alpha = torch.rand(ci.numel(), H, device=DEV, generator=g)
        recv = torch.arange(n, device=DEV).repeat_interleave(rp[1:] - rp[:-1])
        print("L %d %s" % (L, bad), flush=True)

        def forward(f, a):
            return e2f.e2f_wigner6j_conv_forward(ctx, pos, f, rp, ci, a, L, H, 5.0)

        def backward(f, go):
            return e2f.e2f_wigner6j_conv_backward(ctx, pos, f, go, rp, ci, alpha, L, H, 5.0, want_pos=True)

        def same(got, want, hit):
            assert not bool(torch.isfinite(got[hit]).all())
            assert torch.equal(got[~hit], want[~hit]) and bool(torch.isfinite(want).all())

        y = forward(feat, alpha)
        f = feat.clone()
        f[j0, 2, c0] = bad
        hit = torch.zeros_like(y, dtype=torch.bool)
        hit[recv[ci == j0], :, c0] = True
        same(forward(f, alpha), y, hit)
        e = int((ci == j0).nonzero()[0])
        a = alpha.clone()
        a[e, 2] = bad
        hit = torch.zeros_like(y, dtype=torch.bool)
        hit[recv[e], :, 2 * C // H:3 * C // H] = True
        same(forward(feat, a), y, hit)
        gf, ga, gp = backward(feat, gout)
        go = gout.clone()
        go[j0, 2, c0] = bad
        bf, ba, bp = backward(feat, go)
        hit = torch.zeros_like(ga, dtype=torch.bool)
        hit[recv == j0, c0 * H // C] = True
        same(ba, ga, hit)
        hit = torch.zeros_like(gf, dtype=torch.bool)
        hit[ci[recv == j0].long(), :, c0] = True
        same(bf, gf, hit)
        hit = torch.zeros_like(gp, dtype=torch.bool)
        hit[j0] = hit[ci[recv == j0].long()] = True
        same(bp, gp, hit)
    finally:
        ctx.close()


@pytest.mark.parametrize("L", [2, 4, 6])
def test_small_features(L):
    # 2^-100 of the features is 2^-100 of the result, to float rounding: what the
    # split operands lose lies below 2^-133
    import paper_2501_19216_amd as e2f
    ctx = e2f.e2f_create(L, 0)
    try:
        g = torch.Generator(device=DEV).manual_seed(L)
        pos = gpu(syn.quantize(np.random.default_rng(L).uniform(0, 9.0, size=(150, 3))))
        rp, ci = e2f.e2f_neighbor_list(ctx, pos, 5.0)
        feat = torch.randn(150, (L + 1) ** 2, 16, device=DEV, generator=g)
        alpha = torch.rand(ci.numel(), 2, device=DEV, generator=g)
        y, z = (e2f.e2f_wigner6j_conv_forward(ctx, pos, feat * s, rp, ci, alpha, L, 2, 5.0).double() for s in (1.0, 2.0 ** -100))
        err = float((z * 2.0 ** 100 - y).norm() / y.norm())
        print("L %d features of 2^-100: %.2e" % (L, err), flush=True)
        assert err <= 1e-6
    finally:
        ctx.close()


@pytest.mark.parametrize("L,C,H,n,y_norm", [(2, 16, 4, 300, False), (4, 64, 4, 1200, True), (3, 1024, 8, 4003, False)])
def test_forward_under_capture(L, C, H, n, y_norm):
    # a captured forward of a graph that one workgroup plans (receivers in their own
    # order, and sorted: the last case), replayed on new features and positions with
    # eager work in between
    import paper_2501_19216_amd as e2f
    ctx = e2f.e2f_create(L, 0)
    try:
        rng = np.random.default_rng(n)
        pos = gpu(syn.quantize(rng.uniform(0, (n / 0.1) ** (1.0 / 3.0), size=(n, 3))))
        rp, ci = e2f.e2f_knn_graph(ctx, pos, 16)
        g = torch.Generator(device=DEV).manual_seed(n)
        feat = torch.randn(n, (L + 1) ** 2, C, device=DEV, generator=g)
        alpha = torch.rand(ci.numel(), H, device=DEV, generator=g)
        mix = torch.randn(L + 1, C, C, device=DEV, generator=g) / C ** 0.5
        kw = dict(mix_w=mix, y_norm=y_norm)
        e2f.e2f_wigner6j_prepare(ctx, L, C, H, 8.0, **kw)
        size = e2f.e2f_wigner6j_workspace_size(ctx, n, ci.numel(), L, C, H, 8.0, minimum=True, **kw)
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        out = torch.empty_like(feat)

        def forward(o):
            return e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, 8.0, out=o, workspace=ws, **kw)

        forward(out)
        torch.cuda.synchronize()
        print("capture: L %d C %d n %d" % (L, C, n), flush=True)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            forward(out)
        for k in range(4):
            feat.normal_(generator=g)
            pos += 0.25
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            got = out.clone()
            assert torch.equal(got, forward(torch.empty_like(feat))), "replay %d" % k
    finally:
        ctx.close()
