"""The iterations of the field and Gauss-law solves at the places where their
count can go wrong: one iteration, the last allowed one, one too few."""
import numpy as np
import pytest

from paper_2208_12795_amd import synth

pytestmark = pytest.mark.gpu

EPS0, MU0 = 8.8541878128e-12, 1.25663706212e-6
TOL = 1e-12


# one block of rows; ragged blocks; more rows than one block per CU holds
@pytest.fixture(scope="module", params=[(2, 2, 2), (9, 8, 7), (31, 30, 29)], ids=str)
def ctx(request):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2208_12795_amd import etpic as E
    xyz, tv = synth.kuhn_mesh(request.param, (1.0, 1.0, 1.0), 0.1, np.random.default_rng(5))
    c = E.Context(0)
    c.upload_mesh(xyz, tv)
    c.field_setup(2e-11, 3e9, EPS0, MU0)
    c.ns_setup(EPS0)
    yield E, c
    c.close()


def counts_are_kept(E, solve):
    """solve(max_iter) -> (status, iterations, residual, results)"""
    rc, its, res, want = solve(2000)
    assert rc == E.OK and its >= 1 and res <= TOL
    rc, k, r, got = solve(its)
    assert (rc, k, r) == (E.OK, its, res) and np.array_equal(got, want)
    if its > 1:
        for most in sorted({1, its // 2 or 1, its - 1}):
            rc, k, r, _ = solve(most)
            assert rc == E.ENOCONV and k == most and r > TOL
    rc, k, r, got = solve(2000)          # and a solve after one that stopped short
    assert (rc, k, r) == (E.OK, its, res) and np.array_equal(got, want)


def test_field_step_iterations(ctx):
    import torch
    E, c = ctx
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda n: torch.randn((n, 2), dtype=torch.float64, device="cuda", generator=g)
    state = [rnd(c.n_edge), rnd(c.n_edge) * 1e9, rnd(c.n_edge) * 1e18, rnd(c.n_face) * 1e-9]

    def solve(most):
        s = [t.clone() for t in state]
        rc, k, r = c.field_step(2e-11, *s, tol=TOL, max_iter=most, raise_on_error=False)
        return rc, k, r, s[2].cpu().numpy()
    counts_are_kept(E, solve)


def test_gauss_solve_iterations(ctx):
    import torch
    E, c = ctx
    rho0 = torch.randn(c.n_vert, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(2))

    def solve(most):
        e = torch.zeros((c.n_edge, 2), dtype=torch.float64, device="cuda")
        rc, k, r = c.ns_solve(rho0=rho0, e_out=e, tol=TOL, max_iter=most, raise_on_error=False)
        return rc, k, r, e.cpu().numpy()
    counts_are_kept(E, solve)


def test_no_source(ctx):
    import torch
    E, c = ctx
    zero = torch.zeros(c.n_vert, dtype=torch.float64, device="cuda")
    e = torch.ones((c.n_edge, 2), dtype=torch.float64, device="cuda")
    assert c.ns_solve(rho0=zero, e_out=e, tol=TOL) == (E.OK, 0, 0.0)
    assert torch.count_nonzero(e).item() == 0


def test_solves_beside_other_work():
    """Two contexts solving from two threads on streams of their own, beside a
    third stream's products that fill the chip: whichever way a solve takes its
    iterations then, it converges to the result of the quiet one."""
    import threading
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2208_12795_amd import etpic as E
    xyz, tv = synth.kuhn_mesh((20, 20, 20), (1.0, 1.0, 1.0), 0.1, np.random.default_rng(6))
    ctxs = []
    for _ in range(2):
        c = E.Context(0)
        c.upload_mesh(xyz, tv)
        c.field_setup(2e-11, 3e9, EPS0, MU0)
        c.ns_setup(EPS0)
        ctxs.append(c)
    ne, nf, nv = ctxs[0].n_edge, ctxs[0].n_face, ctxs[0].n_vert
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *n: torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    rho0, state = rnd(nv), [rnd(ne, 2), rnd(ne, 2) * 1e9, rnd(ne, 2) * 1e18, rnd(nf, 2) * 1e-9]

    def both(c, stream=None):
        s = [t.clone() for t in state]
        e = torch.zeros((ne, 2), dtype=torch.float64, device="cuda")
        a = c.field_step(2e-11, *s, tol=TOL, stream=stream)
        b = c.ns_solve(rho0=rho0, e_out=e, tol=TOL, stream=stream)
        return a, b, s[2], e
    quiet = both(ctxs[0])
    scale = [float(quiet[k].abs().max()) for k in (2, 3)]
    m = rnd(4096, 4096)
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        for _ in range(8):
            m2 = m @ m
    bad = []

    def work(c):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(4):
                a, b, x, e = both(c, st)
                st.synchronize()
                # both solves stop at a residual of 1e-12: the results differ by that times the condition
                far = max(float((v - q).abs().max()) / s for v, q, s in zip((x, e), quiet[2:], scale))
                if a[0] != E.OK or b[0] != E.OK or abs(a[1] - quiet[0][1]) > 1 or abs(b[1] - quiet[1][1]) > 1 or far > 1e-8:
                    bad.append((a, b, far))
    threads = [threading.Thread(target=work, args=(c,)) for c in ctxs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not bad and bool(torch.isfinite(m2).all())
    for c in ctxs:
        c.close()
