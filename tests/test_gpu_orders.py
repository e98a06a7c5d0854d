"""Block orders of the Wilson operator on lattices whose planes do not hold whole
blocks: eighths of each time slice (also where eight do not divide it) and t
slabs (also with fewer blocks than eight fill), against the plain index order.

The order changes which block computes a site, not how: outputs of one launch
shape are bit-identical; sums of squares are taken over other blocks, in FP64,
so they agree to 1e-13; solutions to 1e-12 on matrices whose smallest
|eigenvalue| is above 1e-2, so 1e-10.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import qcd_inputs as qi  # noqa: E402
from gpu_common import to_dev  # noqa: E402


@pytest.fixture(scope="module")
def q():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2602_14450_amd as q
    return q


@pytest.mark.parametrize("dims,nrhs", [
    ((30, 30, 30, 2), 1),  # eighths that do not divide the slice, all forms
    ((26, 26, 26, 2), 2),  # eighths for the full lattice, t slabs for one parity
    ((32, 24, 16, 2), 3),  # eighths of whole blocks (one parity), whole planes (full lattice)
    ((6, 10, 14, 4), 3),   # t slabs, the last of them short
    ((2, 6, 2, 2), 1),     # one block
])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_orders_agree(q, dims, nrhs, prec):
    k = 0.115
    U = to_dev(qi.gauge_field(dims, 0.3, 501))
    x = to_dev(qi.gaussian_source(dims, 502, nrhs=nrhs))
    g = q.gauge_upload(U, dims)
    for tile in [1] + [t for t in (2, -2, -3) if nrhs % abs(t) == 0]:
        got = []
        for sched in (0, 1, 3):
            for p in (q.FP64, prec):
                g.set_tuning(p, sched, 0, tile)
            outs = [q.dslash(g, k, torch.empty_like(x), x, op=op, prec=prec) for op in (q.OP_D, q.OP_SCHUR)]
            r = torch.empty_like(x)
            norm = np.atleast_1d(q.residual(g, k, r, x, x))
            got.append((outs + [r], norm))
        for outs, norm in got[1:]:
            for a, b in zip(outs, got[0][0]):
                assert torch.equal(a, b), (dims, prec, tile)
            assert np.allclose(norm, got[0][1], rtol=1e-13, atol=0)
    # the reductions of the iterations, over rows of the new orders
    for even_odd in (False, True):
        xs = []
        for sched in (0, 1):
            for p in (q.FP64, prec):
                g.set_tuning(p, sched, 0, 0)
            sol = torch.zeros_like(x)
            if prec == q.FP64:
                info = q.bicgstab(g, k, sol, x, prec=prec, tol=1e-12, even_odd=even_odd)
            else:
                info = q.solve_mixed_ir(g, k, sol, x, inner_prec=prec, tol=1e-12, inner_tol=1e-2, even_odd=even_odd)
            for i in info if isinstance(info, list) else [info]:
                assert i.status == "ok" and i.true_rel_residual <= 1.01e-12
            xs.append(sol)
        assert (xs[0] - xs[1]).norm() <= 1e-10 * xs[1].norm()
    g.close()


@pytest.mark.parametrize("dims,nrhs", [
    ((32, 32, 32, 16), 4),  # four right-hand sides per thread from here on
    ((32, 32, 32, 14), 4),  # two below
])
def test_automatic_tile_agrees(q, dims, nrhs):
    # a thread with several right-hand sides evaluates the same expressions as one
    # with a single one, but a multiply-add may be fused differently: the FP32 sum
    # then rounds to the neighbouring binary16 value at a few outputs
    k = 0.115
    U = to_dev(qi.gauge_field(dims, 0.3, 511))
    x = q.gaussian_spinors((nrhs, 2, int(np.prod(dims)) // 2, 12), 512)
    g = q.gauge_upload(U, dims)
    got = q.dslash(g, k, torch.empty_like(x), x, prec=q.FP16)
    g.set_tuning(q.FP16, 0, 0, 1)
    want = q.dslash(g, k, torch.empty_like(x), x, prec=q.FP16)
    d = (torch.view_as_real(got) - torch.view_as_real(want)).abs()
    assert bool((d <= 2.0 ** -10 * torch.view_as_real(want).abs() + 1e-30).all())
    assert float((d > 0).double().mean()) <= 1e-4
    g.close()
