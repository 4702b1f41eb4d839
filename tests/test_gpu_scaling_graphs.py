"""The graphs of the scaling study (Sec. 4.1 / Fig. 2): the GPU
k-nearest-neighbour graph against the oracle, bit-exact; the Wigner-6j layer
on kNN graphs and on dense graphs (every atom attends to every other) against
the oracle's definition of the layer; uniform attention over the whole graph
(App. G, global moments) against the oracle's global-moment form and, on a
small graph, the definition.

Run with -m gpu."""
import itertools

import numpy as np
import pytest
import torch

import e2f_synth as syn
import oracle as o
from cases import TOL_F32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def e2f():
    import paper_2501_19216_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(e2f):
    c = e2f.e2f_create(6, 0)
    yield c
    c.close()


def gpu(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def knn_both(e2f, ctx, pos, k, gid=None):
    rp, ci = e2f.e2f_knn_graph(ctx, gpu(pos), k, gpu(gid))
    orp, oci = o.knn_graph(pos, k, gid)
    return rp.cpu().numpy(), ci.cpu().numpy(), orp, oci


@pytest.mark.parametrize("n,k,side", [(1000, 32, 21.5), (1000, 512, 21.5), (3000, 8, 31.0), (257, 300, 12.0)])
def test_knn_bit_exact_random(e2f, ctx, n, k, side):
    rng = np.random.default_rng(n + k)
    pos = syn.quantize(rng.uniform(0, side, size=(n, 3)))
    rp, ci, orp, oci = knn_both(e2f, ctx, pos, k)
    print("n %d k %d: %d edges" % (n, k, len(oci)))
    assert np.array_equal(rp, orp) and np.array_equal(ci, oci)


def test_knn_bit_exact_ties_and_graphs(e2f, ctx):
    # a lattice: many equal distances, taken in index order
    g = np.array(list(itertools.product(range(6), repeat=3)), dtype=np.float32) * 1.5
    for k in (6, 7, 18, 20, 26, 64):
        rp, ci, orp, oci = knn_both(e2f, ctx, g, k)
        assert np.array_equal(rp, orp) and np.array_equal(ci, oci), k
    # many small graphs (the 256 x 30 molecules) and a graph of one atom
    inp = syn.make_inputs(syn.WORKLOADS["molecules256x30_L3"])
    gid = inp.graph_id.copy()
    gid[-1] = gid.max() + 1
    for k in (8, 29, 40):
        rp, ci, orp, oci = knn_both(e2f, ctx, inp.pos, k, gid)
        assert np.array_equal(rp, orp) and np.array_equal(ci, oci), k
    assert rp[-1] == rp[-2]  # the lone atom has no neighbours


def knn_inputs(n, k, L, C, H, seed):
    rng = np.random.default_rng(seed)
    side = (n / 0.1) ** (1.0 / 3.0)  # 0.1 atoms / A^3, like the other workloads
    pos = syn.quantize(rng.uniform(0, side, size=(n, 3)))
    rp, ci = o.knn_graph(pos, k)
    d = np.linalg.norm(pos[np.repeat(np.arange(n), np.diff(rp))] - pos[ci], axis=1)
    reach = float(d.max()) * 1.001
    species = rng.integers(0, 10, size=n)
    alpha = syn.attention_weights(pos, species, rp, ci, H, reach, 10, seed)
    feat = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
    return pos, rp, ci, alpha, feat, reach


@pytest.mark.parametrize("n,k,L,C,H,rows", [(600, 32, 3, 64, 8, None), (1000, 256, 3, 32, 4, 96),
                                             (400, 32, 6, 16, 4, 64)])
def test_layer_on_knn_graphs(e2f, ctx, n, k, L, C, H, rows):
    pos, rp, ci, alpha, feat, reach = knn_inputs(n, k, L, C, H, seed=n + k + L)
    w = np.zeros((L + 1) ** 3)
    for a, f, oo in itertools.product(range(L + 1), repeat=3):
        if abs(a - f) <= oo <= a + f:
            w[(a * (L + 1) + f) * (L + 1) + oo] = reach ** (-f)
    r = np.arange(n) if rows is None else np.linspace(0, n - 1, rows).astype(np.int32)
    ref = o.conv_edge(L, H, pos, feat, rp, ci, alpha, w, rows=r)
    for fn in (e2f.e2f_wigner6j_conv_forward, e2f.e2f_edge_tp_conv_forward):
        got = fn(ctx, gpu(pos), gpu(feat), gpu(rp), gpu(ci), gpu(alpha), L, H, reach).cpu().numpy()
        err = o.max_rel_err(got[r], ref, L)
        print("kNN n %d k %d L %d %s: err %.3e" % (n, k, L, fn.__name__, err))
        assert err <= TOL_F32


# ------------------------------------------------------------ dense graphs
def complete_graph(n):
    rp = np.arange(0, n * (n - 1) + 1, n - 1, dtype=np.int64) if n > 1 else np.zeros(n + 1, dtype=np.int64)
    ci = np.array([j for i in range(n) for j in range(n) if j != i], dtype=np.int32)
    return rp, ci


@pytest.mark.parametrize("n,L,C,H,rows,mix", [(160, 3, 32, 4, None, False), (700, 4, 64, 8, 48, True),
                                               (300, 2, 16, 4, None, True)])
def test_dense_graph_layer(e2f, ctx, n, L, C, H, rows, mix):
    rng = np.random.default_rng(n + L)
    side = (n / 0.1) ** (1.0 / 3.0)
    pos = syn.quantize(rng.uniform(0, side, size=(n, 3)))
    feat = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
    A = rng.uniform(0.0, 1.0 / n, size=(n, n, H)).astype(np.float32)
    rp, ci = complete_graph(n)
    alpha = A[np.repeat(np.arange(n), n - 1), ci]  # [E][H] in CSR order
    cutoff = 10.0
    w = np.zeros((L + 1) ** 3)
    for a, f, oo in itertools.product(range(L + 1), repeat=3):
        if abs(a - f) <= oo <= a + f:
            w[(a * (L + 1) + f) * (L + 1) + oo] = cutoff ** (-f)
    mix_w = (rng.standard_normal((L + 1, C, C)) / np.sqrt(C)).astype(np.float32) if mix else None
    r = np.arange(n) if rows is None else np.linspace(0, n - 1, rows).astype(np.int32)
    ref = o.layer(L, H, pos, feat, rp, ci, alpha, w, mix_w, rows=r)
    got = e2f.e2f_wigner6j_conv_forward_dense(ctx, gpu(pos), gpu(feat), gpu(A), L, H, cutoff,
                                              mix_w=gpu(mix_w)).cpu().numpy()
    err = o.max_rel_err(got[r], ref, L)
    print("dense n %d L %d: err %.3e" % (n, L, err))
    assert err <= TOL_F32
    # alpha = None means 1 for every pair
    ones = np.ones((len(ci), H), dtype=np.float32)
    r1 = r[:16]
    ref1 = o.layer(L, H, pos, feat, rp, ci, ones, w, mix_w, rows=r1)
    got1 = e2f.e2f_wigner6j_conv_forward_dense(ctx, gpu(pos), gpu(feat), None, L, H, cutoff,
                                               mix_w=gpu(mix_w)).cpu().numpy()
    assert o.max_rel_err(got1[r1], ref1, L) <= TOL_F32


# The edges of the product's tiles (256 x 128, K slabs of 16, rows of A padded to
# 32, column chunks of 256 and groups of 8 heads).  Float products (split exactly
# into three bf16 parts) and sums of n terms: the layer's bar leaves more than a
# digit over the 1e-6 seen.
@pytest.mark.parametrize("n,L,C,H", [(2, 0, 4, 1), (15, 1, 36, 9), (16, 2, 16, 4), (17, 2, 64, 16), (33, 4, 8, 2),
                                     (64, 3, 12, 3), (255, 1, 8, 1), (257, 2, 40, 10), (289, 3, 32, 8)])
def test_dense_tile_edges(e2f, ctx, n, L, C, H):
    rng = np.random.default_rng(31 * n + L)
    pos = syn.quantize(rng.uniform(0, (n / 0.1) ** (1.0 / 3.0), size=(n, 3)))
    feat = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
    A = rng.uniform(0.0, 1.0 / n, size=(n, n, H)).astype(np.float32)
    rp, ci = complete_graph(n)
    r = np.unique(np.linspace(0, n - 1, 24).astype(np.int32))
    al = A[np.repeat(np.arange(n), n - 1), ci]
    print("dense n %d L %d C %d H %d" % (n, L, C, H), flush=True)
    for weights, ref_al in ((gpu(A), al), (None, np.ones_like(al))):
        got = e2f.e2f_wigner6j_conv_forward_dense(ctx, gpu(pos), gpu(feat), weights, L, H, 10.0).cpu().numpy()
        err = o.max_rel_err(got[r], o.layer(L, H, pos, feat, rp, ci, ref_al, default_w(L, 10.0), rows=r), L)
        print("  err %.3e" % err)
        assert err <= TOL_F32


def test_dense_graph_single_atom(e2f, ctx):
    feat = np.ones((1, 9, 8), dtype=np.float32)
    got = e2f.e2f_wigner6j_conv_forward_dense(ctx, gpu(np.zeros((1, 3), np.float32)), gpu(feat),
                                              gpu(np.ones((1, 1, 2), np.float32)), 2, 2, 5.0).cpu().numpy()
    assert np.all(got == 0)


# ------------------------------------------------------------ global moments (App. G)
def default_w(L, cutoff):
    w = np.zeros((L + 1) ** 3)
    for a, f, oo in itertools.product(range(L + 1), repeat=3):
        if abs(a - f) <= oo <= a + f:
            w[(a * (L + 1) + f) * (L + 1) + oo] = cutoff ** (-f)
    return w


@pytest.mark.parametrize("n,L,C,H,rows,mix", [(200, 2, 16, 4, None, False), (1500, 4, 64, 8, 64, True),
                                               (400, 6, 16, 2, 32, False), (5000, 4, 128, 8, 24, False),
                                               (333, 3, 12, 3, None, True)])
def test_global_moment_layer(e2f, ctx, n, L, C, H, rows, mix):
    rng = np.random.default_rng(7 * n + L)
    side = (n / 0.1) ** (1.0 / 3.0)
    pos = syn.quantize(rng.uniform(0, side, size=(n, 3)))
    feat = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
    cutoff = 10.0
    w = default_w(L, cutoff)
    mix_w = (rng.standard_normal((L + 1, C, C)) / np.sqrt(C)).astype(np.float32) if mix else None
    r = np.arange(n, dtype=np.int32) if rows is None else np.linspace(0, n - 1, rows).astype(np.int32)
    y = o.conv_global(L, pos, feat, w, pos.astype(np.float64).mean(0), rows=r)
    ref = y if mix_w is None else o.mix(L, y, mix_w)
    print("global n %d L %d C %d: case" % (n, L, C), flush=True)
    got = e2f.e2f_wigner6j_conv_forward_global(ctx, gpu(pos), gpu(feat), L, H, cutoff,
                                               mix_w=gpu(mix_w)).cpu().numpy()
    err = o.max_rel_err(got[r], ref, L)
    print("global n %d L %d: err %.3e" % (n, L, err))
    assert err <= TOL_F32
    # default path weights are cutoff^-f on the triangle-valid paths
    got_d = e2f.e2f_wigner6j_conv_forward_global(ctx, gpu(pos), gpu(feat), L, H, cutoff, path_w=None,
                                                 mix_w=gpu(mix_w)).cpu().numpy()
    assert np.array_equal(got_d, got)


def test_global_moment_equals_definition(e2f, ctx):
    # the definition on the complete graph with self edges and alpha = 1
    n, L, C, H = 90, 3, 8, 2
    rng = np.random.default_rng(5)
    pos = syn.quantize(rng.uniform(0, 9.0, size=(n, 3)))
    feat = rng.standard_normal((n, (L + 1) ** 2, C)).astype(np.float32)
    w = default_w(L, 5.0)
    rp = np.arange(n + 1, dtype=np.int64) * n
    ci = np.tile(np.arange(n, dtype=np.int32), n)
    ref = o.layer(L, H, pos, feat, rp, ci, np.ones((n * n, H), np.float32), w)
    got = e2f.e2f_wigner6j_conv_forward_global(ctx, gpu(pos), gpu(feat), L, H, 5.0).cpu().numpy()
    err = o.max_rel_err(got, ref, L)
    print("global vs definition: err %.3e" % err)
    assert err <= TOL_F32
    # one atom: only its self term, R^(f)(0) = [f == 0]
    one = e2f.e2f_wigner6j_conv_forward_global(ctx, gpu(pos[:1]), gpu(feat[:1]), L, H, 5.0).cpu().numpy()
    ref1 = o.layer(L, H, pos[:1], feat[:1], np.array([0, 1], np.int64), np.zeros(1, np.int32),
                   np.ones((1, H), np.float32), w)
    assert o.max_rel_err(one, ref1, L) <= TOL_F32
    # deterministic: a second call gives the same bits
    again = e2f.e2f_wigner6j_conv_forward_global(ctx, gpu(pos), gpu(feat), L, H, 5.0).cpu().numpy()
    assert np.array_equal(again, got)
