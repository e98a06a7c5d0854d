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

import oracle  # noqa: E402
import qcd_inputs as qi  # noqa: E402
from gpu_common import TOL, compare, to_dev, to_host  # noqa: E402


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


# rounding of a result from the same products in the same order, where the
# compiler may fuse a sum differently: one unit of 16-bit storage (two after the
# two hops of the Schur operator); in 32 and 64 bits a few units of the sums' terms
UNIT = {0: 2.0 ** -52, 1: 2.0 ** -23, 2: 2.0 ** -10, 3: 2.0 ** -7}


@pytest.mark.parametrize("dims", [
    (16, 48, 18, 4),   # full lattice: 54 blocks of three planes' x rows over eight XCDs
    (32, 40, 10, 4),   # full lattice: 50 blocks
    (16, 32, 36, 4),   # one parity: 36 blocks; the full lattice past 8 planes a sub-slab
    (32, 16, 30, 8),   # one parity: 30 blocks
])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_lds_forms_in_the_orders_of_ragged_slices(q, dims, prec):
    # planes of whole blocks and Lz no multiple of 8: the untouched handle and the
    # LDS variants against index order without LDS, and against the oracle
    k = 0.115
    U, b = qi.gauge_field(dims, 0.3, 521), qi.gaussian_source(dims, 522)
    g = q.gauge_upload(to_dev(U), dims)
    x = to_dev(b)
    shapes = [(sched, v, 1) for sched in (1, 2) for v in (6, 7)]
    ops = (q.OP_D, q.OP_H, q.OP_DDAG, q.OP_SCHUR)

    def run():
        return [torch.view_as_real(q.dslash(g, k, torch.empty_like(x), x, op=op, prec=prec)) for op in ops]

    got = [run()]  # the default shape
    for s in shapes:
        g.set_tuning(prec, *s)
        got.append(run())
    g.set_tuning(prec, 0, 0, 1)
    want = run()
    compare(to_host(want[0]), np.ascontiguousarray(oracle.dslash(U, b, k, dims)).view(np.float64), TOL[prec], "oracle")
    for outs in got:
        for op, a, w in zip(ops, outs, want):
            d = (a - w).abs()
            if prec >= 2:
                assert bool((d <= 2 * UNIT[prec] * w.abs() + 1e-30).all()), (dims, prec, op)
                assert float((d > 0).double().mean()) <= 1e-2, (dims, prec, op)
            else:
                assert float(d.max()) <= 16 * UNIT[prec] * float(w.square().mean().sqrt()), (dims, prec, op)
    # the one-parity reductions and the residual's sum
    for s in [None] + shapes[:2]:
        for p in (q.FP64, prec):
            if s:
                g.set_tuning(p, *s)
        sol = torch.zeros_like(x)
        if prec == q.FP64:
            info = q.bicgstab(g, k, sol, x, prec=prec, tol=1e-12, even_odd=True)
        else:
            info = q.solve_mixed_ir(g, k, sol, x, inner_prec=prec, tol=1e-12, inner_tol=1e-2, even_odd=True)
        r = torch.empty_like(x)
        norm = q.residual(g, k, r, sol, x)
        assert info.status == "ok" and info.true_rel_residual <= 1.01e-12
        # the residual of the solution, summed by torch
        assert abs(norm - float(r.abs().square().sum())) <= 1e-12 * norm
        res = np.linalg.norm(b - oracle.dslash(U, to_host(sol), k, dims)) / np.linalg.norm(b)
        assert res <= 1.01e-12, (dims, prec, s, res)
    g.close()
