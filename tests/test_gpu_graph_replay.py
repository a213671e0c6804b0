"""Step calls recorded into a HIP graph: every replay, with the context's own
eager calls in between, gives what the eager call gives."""
import numpy as np
import pytest

from paper_2208_12795_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind,nsteps", [("step", 1), ("run", 10), ("run", 20), ("forced", 3), ("downshifted", 1),
                                         ("downshifted", 10)])
def test_replays_equal_eager_calls(kind, nsteps, precision):
    """Identical particles; the current to the rounding of its sums (1e-13 of
    the largest, as in the tests of several steps per launch)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2208_12795_amd import etpic as E
    w = synth.make_workload(1, n_particles=5000)
    o = np.argsort(w.tet, kind="stable")
    ctx = E.Context(0)
    ctx.upload_mesh(w.xyz, w.tet_vert)
    f = E.Fields.from_numpy(w.e_env, 1e-3 * w.b_env, None, 1e-3 * w.b_dc)
    sp = E.Species(w.q, w.m, w.w)
    p0 = E.Particles.from_numpy(w.tet[o], w.lam[o], w.vel[o], w.ids[o], precision=precision)
    p0.vel *= 30.0
    dt = 30.0 * w.dt
    p, g = p0.clone(), torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    hist = ctx.ds_history(p)

    def call(p, g, hist):
        if kind == "step":
            ctx.gather_push_deposit(p, sp, f, 7, dt, w.omega, g)
        elif kind == "downshifted":
            ctx.ds_steps(p, hist, sp, f, 7, nsteps, 0, dt, w.omega, g)
        else:
            ctx.run_steps(p, sp, f, 7, nsteps, dt, w.omega, g,
                          flags=E.STEP_XCD_REMAP | (E.STEP_SLICES_4 if kind == "forced" else 0))

    def eager():
        q, h = p0.clone(), torch.zeros_like(g)
        call(q, h, torch.zeros_like(hist))
        return q, h
    want, g_want = eager()     # (also binds the downshifted rows before the recording)
    ctx.check()
    assert (want.tet != p0.tet).double().mean().item() > 0.01 or nsteps < 10
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(p, g, hist)
    for replay in range(5):
        for a, b in ((p.lam, p0.lam), (p.vel, p0.vel), (p.tet, p0.tet)):
            a.copy_(b)
        g.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in ((p.lam, want.lam), (p.vel, want.vel), (p.tet, want.tet)):
            assert torch.equal(a, b)
        assert torch.allclose(g, g_want, rtol=0, atol=1e-13 * g_want.abs().max().item()), replay
        if replay == 2:
            q, h = eager()
            assert torch.equal(q.tet, want.tet)
            assert torch.allclose(h, g_want, rtol=0, atol=1e-13 * g_want.abs().max().item())
    ctx.check()
    ctx.close()
