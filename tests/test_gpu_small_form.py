"""The small-lattice forms (one hop per wave; the folded even-odd and full
iterations) against the forms that a set launch shape selects, at the edges of
their range: lattices below one 64-site block, ragged last blocks, exactly the
largest call and just past it, several right-hand sides.

Tolerances: those of the operator tests against the oracle (gpu_common.TOL:
rounding of the sums' order, one storage rounding in 16 bits); solutions to
1e-12 on matrices whose smallest |eigenvalue| is above 1e-2, so 1e-10, and
iteration counts that may move by one where a stop is met at its edge.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import qcd_inputs as qi  # noqa: E402
from gpu_common import TOL, compare, to_dev, to_host  # noqa: E402

SHAPES = {0: (1, 0, 1), 1: (1, 6, 1), 2: (1, 6, 1), 3: (1, 1, 1)}


@pytest.fixture(scope="module")
def q():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2602_14450_amd as q
    return q


@pytest.mark.parametrize("dims,nrhs,full_links", [
    ((2, 2, 2, 2), 1, False),      # 8 sites per parity
    ((2, 4, 6, 10), 3, True),      # 240 sites per parity, 18 reals per link
    ((8, 16, 16, 16), 1, False),   # 512 blocks: the largest full-lattice call in 16 and 32 bits
    ((8, 16, 16, 18), 1, False),   # past it
    ((16, 16, 16, 16), 1, False),  # one parity at its limit, the full lattice past it
])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_operator_forms_agree(q, dims, nrhs, full_links, prec):
    U = qi.gauge_field(dims, 0.3, 301)
    psi = qi.gaussian_source(dims, 302, nrhs=nrhs)
    k = 0.12
    g = q.gauge_upload(to_dev(U), dims, full_links=full_links)
    x = to_dev(psi)
    got = {op: to_host(q.dslash(g, k, torch.empty_like(x), x, op=op, prec=prec)) for op in (0, 1, 2, 3, 4)}
    g.set_tuning(prec, *SHAPES[prec])
    for op in got:
        want = to_host(q.dslash(g, k, torch.empty_like(x), x, op=op, prec=prec))
        compare(got[op], want, TOL[prec], f"op {op} prec {prec} dims {dims}")
    for r in range(nrhs):
        compare(got[0][r], oracle.dslash(U, psi[r], k, dims), TOL[prec], f"oracle, right-hand side {r}")
    g.close()


@pytest.mark.parametrize("dims,nrhs", [((2, 4, 6, 10), 2), ((4, 4, 4, 8), 1), ((8, 8, 8, 8), 3)])
@pytest.mark.parametrize("even_odd", [False, True])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_folded_solves_agree(q, dims, nrhs, even_odd, prec):
    k = 0.115
    U = qi.gauge_field(dims, 0.3, 311)
    b = to_dev(qi.gaussian_source(dims, 312, nrhs=nrhs))
    if nrhs > 2:
        b[1] = 0  # a right-hand side that stops before the first iteration
    g = q.gauge_upload(to_dev(U), dims)
    runs = []
    for shaped in (False, True):
        if shaped:
            for p in SHAPES:
                g.set_tuning(p, *SHAPES[p])
        x = torch.zeros_like(b)
        if prec == q.FP64:
            info = q.bicgstab(g, k, x, b, prec=prec, tol=1e-12, even_odd=even_odd, sigma=64.0, sigma_lambda=64.0)
        else:
            info = q.solve_mixed_ir(g, k, x, b, inner_prec=prec, tol=1e-12, inner_tol=1e-2, even_odd=even_odd)
        runs.append((to_host(x), info if isinstance(info, list) else [info]))
    (x0, i0), (x1, i1) = runs
    for r in range(nrhs):
        assert i0[r].status == "ok" and i0[r].true_rel_residual <= 1.01e-12
        assert abs(i0[r].inner_iters - i1[r].inner_iters) <= 1 + i1[r].outer_iters, (i0[r], i1[r])
        scale = max(np.linalg.norm(x1[r]), 1e-300)
        assert np.linalg.norm(x0[r] - x1[r]) <= 1e-10 * scale
    # a step cap: the folded iteration stops where it should
    x = torch.zeros_like(b)
    capped = q.bicgstab(g, k, x, b, prec=prec, tol=1e-30, max_iter=3, even_odd=even_odd)
    for i in capped if isinstance(capped, list) else [capped]:
        assert i.inner_iters <= 3
    g.close()


@pytest.mark.parametrize("dims", [(12, 12, 12, 12), (8, 16, 16, 16)])
@pytest.mark.parametrize("even_odd", [False, True])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_folded_solves_do_not_depend_on_the_chunks(q, dims, even_odd, prec):
    # more partial rows than the folded kernels have threads: where the host cuts
    # its chunks of iterations (check_every, or what a solve before showed) does
    # not reach the sums, so every run has the same bits
    k = 0.115
    g = q.gauge_upload(to_dev(qi.gauge_field(dims, 0.3, 321)), dims)
    b = to_dev(qi.gaussian_source(dims, 322))
    runs = []
    for every in (0, 0, 1, 5):
        x = torch.zeros_like(b)
        i = q.bicgstab(g, k, x, b, prec=prec, tol=1e-12 if prec == q.FP64 else 1e-2, even_odd=even_odd,
                       check_every=every)
        assert i.status == "ok"
        runs.append((to_host(x), np.asarray(i.history), i.inner_iters))
    if prec != q.FP64:
        for every in (0, 0, 2):  # 0: the device takes the refinement steps, 2: the host
            x = torch.zeros_like(b)
            i = q.solve_mixed_ir(g, k, x, b, inner_prec=prec, tol=1e-12, inner_tol=1e-2, even_odd=even_odd,
                                 check_every=every)
            assert i.status == "ok"
            runs.append((to_host(x), np.zeros(0), i.inner_iters))
    for first, group in ((0, runs[1:4]), (4, runs[5:])):
        for x, history, iters in group:
            assert iters == runs[first][2]
            assert np.array_equal(history, runs[first][1])
            assert np.array_equal(x, runs[first][0])
    g.close()


@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 1), ((8, 16, 16, 16), 2), ((16, 16, 16, 16), 1)])
def test_folded_iterations_take_no_workspace_of_their_own(q, dims, nrhs):
    # vectors, history, eight FP64 sums per partial row (of the kernel with the most
    # rows: 1024, or one per 256 granules of an FP64 field), and the scalars
    g = q.gauge_upload(to_dev(qi.gauge_field(dims, 0.3, 351)), dims)
    vh, max_iter = int(np.prod(dims)) // 2, 1000

    def take(*sizes):
        return sum((s + 255) // 256 * 256 for s in sizes)

    rows = min(1024, 2 * vh * 12 // 256)
    small = [8 * max_iter * nrhs, 64 * rows * nrhs, 64 * nrhs, 8 * nrhs]
    for prec, size in ((q.FP64, 16), (q.FP32, 8), (q.FP16, 4)):
        scalars = 512 * nrhs  # at most
        one, field64 = vh * 12 * size * nrhs, vh * 12 * 16 * nrhs
        eo = take(*[field64] * 7, *[one] * 7, *small)
        full = take(*[2 * field64] * 3, *[2 * one] * 6, *small)
        for what, want in ((9, eo), (1, full)):
            got = g.workspace_bytes(what, prec, max_iter, nrhs)
            assert want <= got <= want + take(scalars), (what, prec, got - want)
    g.close()


def test_launch_shapes_give_the_small_form_back(q, tmp_path):
    # FP64 adds its hops in another order in the small-lattice form, so the bits
    # of a result tell the forms apart
    dims, k, cache = (8, 8, 8, 8), 0.12, str(tmp_path / "tune.jsonl")
    U = to_dev(qi.gauge_field(dims, 0.3, 331))
    x = to_dev(qi.gaussian_source(dims, 332))
    g = q.gauge_upload(U, dims)

    def runs(h):
        return [q.dslash(h, k, torch.empty_like(x), x, op=op, prec=q.FP64) for op in (q.OP_D, q.OP_SCHUR)]

    def same(a, b):
        return all(torch.equal(s, t) for s, t in zip(a, b))

    small, untouched = runs(g), g.get_tuning(q.FP64)
    g.set_tuning(q.FP64, *untouched)  # what the handle has: no change
    assert same(runs(g), small)
    g.set_tuning(q.FP64, *SHAPES[0])
    plain = runs(g)
    assert not torch.equal(plain[0], small[0]) and not torch.equal(plain[1], small[1])
    g.set_tuning(q.FP64, *untouched)
    assert same(runs(g), small)
    # the tuner times the small form too (here 4.0 us against 8.1); another shape
    # drops its choice, the values that it returned and the cache bring it back
    tuned = g.autotune(q.FP64, nrhs=1, reps=50, cache_path=cache)[:3]
    assert same(runs(g), small)
    other = SHAPES[0] if tuned != SHAPES[0] else (0, 0, 1)
    g.set_tuning(q.FP64, *other)
    assert same(runs(g), plain)
    g.set_tuning(q.FP64, *tuned)
    assert same(runs(g), small)
    h = q.gauge_upload(U, dims)
    h.set_tuning(q.FP64, *other)
    assert h.autotune(q.FP64, nrhs=1, cache_path=cache)[:3] == tuned and same(runs(h), small)
    h.close()
    g.close()


def test_tuned_shape_keeps_the_small_one_parity_form(q, tmp_path):
    # 16^4: the full-lattice operator, which the tuner times, is past the small
    # form's range and the one-parity launches are within it
    dims, k, cache = (16, 16, 16, 16), 0.12, str(tmp_path / "tune.jsonl")
    U = to_dev(qi.gauge_field(dims, 0.3, 341))
    x = to_dev(qi.gaussian_source(dims, 342))
    g = q.gauge_upload(U, dims)

    def schur(h):
        return q.dslash(h, k, torch.empty_like(x), x, op=q.OP_SCHUR, prec=q.FP64)

    small = schur(g)
    tuned = g.autotune(q.FP64, nrhs=1, reps=5, cache_path=cache)[:3]
    assert torch.equal(schur(g), small)
    g.set_tuning(q.FP64, *(SHAPES[0] if tuned != SHAPES[0] else (0, 0, 1)))
    assert not torch.equal(schur(g), small)  # a shape that is set holds for every launch
    g.set_tuning(q.FP64, *tuned)
    assert torch.equal(schur(g), small)
    h = q.gauge_upload(U, dims)
    h.autotune(q.FP64, nrhs=1, cache_path=cache)
    assert torch.equal(schur(h), small)
    h.close()
    g.close()
