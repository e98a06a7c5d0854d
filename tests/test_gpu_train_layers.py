"""The network's training layers (X formed in LDS, 64 sites at a time) against the
FP64 oracle where their tiling can go wrong: lattices smaller than one 64-site
block, ragged last blocks, batches that do not divide over the eight XCDs,
every (C_in, C_out) pair, both link storages, and enough site blocks that a
block of the weight gradient walks several of them and flushes its FP32 sums.

Tolerance: that of the BF16 gradients in test_gpu_ptc (products of BF16-rounded
factors, unit roundoff 2^-9, through at most three layers and their
back-propagation): 1e-2 for the loss, 3e-2 in norm per layer.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import qcd_inputs as qi  # noqa: E402
from oracle import ptc as P  # noqa: E402
from gpu_common import to_dev  # noqa: E402


@pytest.mark.parametrize("dims,channels,batch,full_links", [
    ((2, 2, 2, 2), (1, 1, 1), 1, False),       # 8 sites per parity, one item per XCD at most
    ((2, 4, 6, 10), (1, 2, 1, 1), 3, False),   # 240 sites per parity: 3 blocks and 48 sites
    ((6, 4, 4, 6), (1, 1, 2, 1), 5, True),     # 288 sites per parity, 18 reals per link
    ((4, 4, 4, 8), (1, 2, 2, 1), 17, False),
    ((8, 8, 8, 8), (1, 2, 2, 1), 36, False),   # 2304 items: up to five per weight-gradient block
])
def test_training_layers_match_oracle(dims, channels, batch, full_links):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2602_14450_amd as q
    k = 0.12
    U = qi.gauge_field(dims, 0.3, 170)
    base = min(batch, 2)
    rs = qi.gaussian_source(dims, 171, nrhs=base)
    es = qi.gaussian_source(dims, 172, nrhs=base)
    Ws = qi.ptc_weights(channels, seed=173, scale=0.5)
    nb = P.neighbours(dims)
    # the batch repeats the base sources; their weights in the mean follow
    slots = [i % base for i in range(batch)]
    share = [slots.count(i) / batch for i in range(base)]
    g = q.gauge_upload(to_dev(U), dims, full_links=full_links)
    net = q.PTC(g, channels, max_batch=batch)
    net.set_weights(Ws)
    r_d, e_d = to_dev(rs[slots]), to_dev(es[slots])
    for got, one in ((net.loss_grad(r_d, e_d), lambda i: P.grad(U, [rs[i]], [es[i]], Ws, nb)),
                     (net.loss_grad_residual(k, r_d), lambda i: P.grad_residual(U, k, [rs[i]], Ws, nb, dims))):
        parts = [one(i) for i in range(base)]
        want_loss = sum(w * p[0] for w, p in zip(share, parts))
        assert abs(got[0] - want_loss) <= 1e-2 * want_loss, (got[0], want_loss)
        for l, gr in enumerate(got[1]):
            want = sum(w * p[1][l] for w, p in zip(share, parts))
            r = np.linalg.norm(gr - want) / np.linalg.norm(want)
            assert r <= 3e-2, f"layer {l}: gradient norm-relative error {r:.3e}"
    net.close()
    g.close()


@pytest.mark.parametrize("dims,channels", [((6, 6, 6, 6), (1, 2, 2, 1)), ((2, 4, 6, 10), (1, 2, 1, 1))])
def test_gradient_after_a_non_finite_one(dims, channels):
    # ragged last blocks: a batch whose gradient is not finite leaves nothing that
    # a later finite batch reads, of the same size or a smaller one
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2602_14450_amd as q
    k, batch = 0.12, 8
    r = to_dev(qi.gaussian_source(dims, 181, nrhs=batch))
    bad = torch.full_like(r, complex(float("nan"), float("inf")))
    g = q.gauge_upload(to_dev(qi.gauge_field(dims, 0.3, 180)), dims)
    ws = qi.ptc_weights(channels, seed=182, scale=0.5)

    def net():
        n = q.PTC(g, channels, max_batch=batch)
        n.set_weights(ws)
        return n

    used = net()
    for n in (batch, 5, 2, 1):
        used.loss_grad_residual(k, bad)
        loss, grad = used.loss_grad_residual(k, r[:n].contiguous())
        fresh = net()
        want_loss, want = fresh.loss_grad_residual(k, r[:n].contiguous())
        fresh.close()
        assert np.isfinite(loss) and loss == want_loss, n
        for l, (a, b) in enumerate(zip(grad, want)):
            assert np.array_equal(a, b), (n, l, np.isfinite(a).all())
    used.close()
    g.close()


def test_weight_gradient_sums_are_short():
    # one source: each 64-site block holds one large value and its negative, in
    # other colours, among ones.  An FP32 chain that spans both loses the ones
    # between them (the unit in the last place of 2^30 is 128); chains of 32 columns
    # lose at most the 31 that share theirs with either, of 190
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2602_14450_amd as q
    dims = (8, 8, 8, 8)
    V = int(np.prod(dims))
    r = np.zeros((V, 4, 3), dtype=np.complex128)
    r[:, :2, :] = 1
    at = (np.arange(V) // 2) % 64 == 0  # the first site of every block of either parity
    r[at, 0, 0], r[at, 0, 2] = 2.0 ** 30, -2.0 ** 30
    e = np.zeros_like(r)
    e[:, 0, :] = 1
    g = q.gauge_upload(to_dev(np.broadcast_to(np.eye(3, dtype=np.complex128), (V, 4, 3, 3)).copy()), dims)
    net = q.PTC(g, (1, 1), max_batch=1)
    net.set_weights([np.zeros((9, 1, 1, 4, 4), dtype=np.complex128)])
    w = net.loss_grad(to_dev(r), to_dev(e))[1][0][0, 0, 0]
    share = (w[0, 0] / w[0, 1]).real  # of the 192 products of a block
    assert (190 - 62) / 192 <= share <= (190 + 62) / 192, share
    net.close()
    g.close()
