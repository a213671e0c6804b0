"""Several steps per launch (etpic_run_steps, etpic_sort_run_steps,
etpic_coarse_step) at the sizes where the split of the work can go wrong:
one particle, wavefronts and blocks that end on a ragged slice, wavefronts
whose particles sit in more tets than are staged at a time, more steps than
one launch takes, particles that leave their tet at every step of a launch."""
import numpy as np
import pytest

from paper_2208_12795_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def E():
    from paper_2208_12795_amd import etpic
    return etpic


def problem(E, torch, n, precision, ordered):
    w = synth.make_workload(1, n_particles=n)
    if ordered:
        o = np.argsort(w.tet, kind="stable")
        w.tet, w.lam, w.vel, w.ids = w.tet[o], w.lam[o], w.vel[o], w.ids[o]
    ctx = E.Context(0)
    ctx.upload_mesh(w.xyz, w.tet_vert)
    f = E.Fields.from_numpy(w.e_env, w.b_env, None, w.b_dc)
    return w, ctx, f, E.Species(w.q, w.m, w.w), E.Particles.from_numpy(w.tet, w.lam, w.vel, w.ids, precision=precision)


def same_state(a, b):
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)


# 32768 and 32769: the last size with 16 particles to a wavefront and the first with 64
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n,ordered,nsteps,dt_scale,by_slice", [
    (1, True, 2, 1.0, False), (63, False, 16, 1.0, False), (65, False, 17, 300.0, False),
    (1000, False, 33, 1000.0, False), (1000, True, 16, 1000.0, True), (32768, False, 3, 300.0, False),
    (32769, False, 3, 300.0, False), (32769, True, 16, 300.0, True), (100_003, True, 10, 1.0, False)])
def test_multi_equals_single_steps(E, torch_cuda, n, ordered, nsteps, dt_scale, by_slice, precision):
    """One call of nsteps against nsteps calls of one step: identical particles;
    currents and charge to the rounding of their sums (1e-13 of the largest,
    the tolerance of the other tests of this identity)."""
    torch = torch_cuda
    w, ctx, f, sp, p1 = problem(E, torch, n, precision, ordered)
    p2 = p1.clone()
    dt = w.dt * dt_scale
    flags = E.STEP_XCD_REMAP | (E.STEP_WALK_BY_SLICE if by_slice else 0)
    g1 = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    g2 = torch.zeros_like(g1)
    rho1 = torch.zeros(ctx.n_vert, dtype=torch.float64, device="cuda")
    rho2 = torch.zeros_like(rho1)
    ctx.run_steps(p1, sp, f, 7, nsteps, dt, w.omega, g1, rho=rho1, flags=flags)
    for j in range(nsteps):
        ctx.gather_push_deposit(p2, sp, f, 7 + j, dt, w.omega, g2, rho=rho2 if j == nsteps - 1 else None, flags=flags)
    ctx.check()
    same_state(p1.to_numpy(), p2.to_numpy())
    if dt_scale > 1:
        moved = (p1.tet.cpu().numpy() != w.tet).mean()
        print(f"[multi] moved to another tet: {moved:.3f}", flush=True)
        assert moved > 0.01
    assert torch.allclose(g1, g2, rtol=0, atol=1e-13 * g2.abs().max().item())
    assert torch.allclose(rho1, rho2, rtol=0, atol=1e-13 * rho2.abs().max().item())
    ctx.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n,ordered,nsteps,dt_scale", [(1, True, 2, 1.0), (1000, False, 18, 300.0),
                                                       (40_001, True, 10, 300.0)])
def test_sorting_multi_equals_sort_then_single_steps(E, torch_cuda, n, ordered, nsteps, dt_scale, precision):
    torch = torch_cuda
    w, ctx, f, sp, src = problem(E, torch, n, precision, ordered)
    dt = w.dt * dt_scale
    d1, d2 = src.empty_like(), src.empty_like()
    g1 = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    g2 = torch.zeros_like(g1)
    ctx.sort_run_steps(src, d1, sp, f, 0, nsteps, dt, w.omega, g1)
    ctx.sort(src, d2)
    for j in range(nsteps):
        ctx.gather_push_deposit(d2, sp, f, j, dt, w.omega, g2)
    ctx.check()
    a, b = d1.to_numpy(), d2.to_numpy()
    oa, ob = np.argsort(a[3]), np.argsort(b[3])
    same_state([x[oa] for x in a], [x[ob] for x in b])
    assert torch.allclose(g1, g2, rtol=0, atol=1e-13 * g2.abs().max().item())
    ctx.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n,ordered", [(65, False), (40_001, True)])
def test_coarse_launch_split_changes_nothing(E, torch_cuda, n, ordered, precision):
    """Twenty fine steps with three different snapshots (two launches) against
    the same call with its slices forced to one, which takes one step per
    launch."""
    torch = torch_cuda
    w, ctx, f, sp, p1 = problem(E, torch, n, precision, ordered)
    snaps = [E.Fields.from_numpy(e, b, None, w.b_dc) for e, b in synth.envelope_snapshots(w, seed=3)]
    p2 = p1.clone()
    g1 = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    g2 = torch.zeros_like(g1)
    dtc = 20 * 300.0 * w.dt
    ctx.coarse_step(p1, sp, snaps, 3 * dtc, dtc, 20, w.omega, g1)
    ctx.coarse_step(p2, sp, snaps, 3 * dtc, dtc, 20, w.omega, g2, flags=E.STEP_XCD_REMAP | E.STEP_SLICES_1)
    ctx.check()
    same_state(p1.to_numpy(), p2.to_numpy())
    assert torch.allclose(g1, g2, rtol=0, atol=1e-13 * g2.abs().max().item())
    ctx.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,ordered,nsteps,dt_scale,edc,by_slice", [
    (1, True, 5, 1.0, False, False), (65, False, 20, 100.0, True, False), (1000, False, 21, 100.0, False, True),
    (40_001, True, 13, 100.0, True, False)])
def test_downshifted_launch_split_changes_nothing(E, torch_cuda, n, ordered, nsteps, dt_scale, edc, by_slice, precision):
    """One call from an empty history (three one-step launches, then up to 16
    steps each) against one call per step: identical particles and history,
    currents and charge to the rounding of their sums."""
    torch = torch_cuda
    w, ctx, _, sp, p1 = problem(E, torch, n, precision, ordered)
    # a weak magnetic field: the explicit multistep scheme is stable at these
    # steps, long enough for particles to cross faces
    f = E.Fields.from_numpy(w.e_env, 1e-3 * w.b_env, 0.3 * w.e_env.real if edc else None, 1e-3 * w.b_dc)
    p1.vel *= 30.0 if dt_scale > 1 else 1.0
    p2 = p1.clone()
    h1, h2 = ctx.ds_history(p1), ctx.ds_history(p2)
    dt = w.dt * dt_scale
    flags = E.STEP_XCD_REMAP | (E.STEP_WALK_BY_SLICE if by_slice else 0)
    g1 = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    g2 = torch.zeros_like(g1)
    rho1 = torch.zeros(ctx.n_vert, dtype=torch.float64, device="cuda")
    rho2 = torch.zeros_like(rho1)
    ctx.ds_steps(p1, h1, sp, f, 6, nsteps, 0, dt, w.omega, g1, rho=rho1, flags=flags)
    for j in range(nsteps):
        ctx.ds_steps(p2, h2, sp, f, 6 + j, 1, j, dt, w.omega, g2, rho=rho2 if j == nsteps - 1 else None, flags=flags)
    ctx.check()
    same_state(p1.to_numpy(), p2.to_numpy())
    if dt_scale > 1:
        moved = (p1.tet.cpu().numpy() != w.tet).mean()
        print(f"[multi] moved to another tet: {moved:.3f}", flush=True)
        assert moved > 0.01
    assert torch.equal(h1, h2)
    assert torch.allclose(g1, g2, rtol=0, atol=1e-13 * g2.abs().max().item())
    assert torch.allclose(rho1, rho2, rtol=0, atol=1e-13 * rho2.abs().max().item())
    ctx.close()


@pytest.mark.parametrize("n,nsteps,every,speed", [(1, 3, 2, 1.0), (65, 12, 7, 30.0), (1000, 11, 11, 30.0), (40_001, 6, 6, 30.0)])
def test_reverse_in_pieces_matches_every_step_checkpoints(E, torch_cuda, n, nsteps, every, speed):
    """The reverse sweep takes up to five steps per launch and recomputes the
    states its later pieces start from: against the sweep with a checkpoint
    before every step (one step per launch), and the forward state against
    single steps; the same sums in another order, so 1e-12 of the largest
    entry (about nsteps orders of the rounding of a step)."""
    torch = torch_cuda
    w, ctx, f, sp, p0 = problem(E, torch, n, 0, n > 1000)
    p0.vel *= speed
    dt = 1e-9
    out = []
    for ev in (every, 1):
        p = p0.clone()
        ws = torch.empty(ctx.adjoint_workspace_bytes(n, nsteps, ev), dtype=torch.uint8, device="cuda")
        ctx.forward_checkpointed(p, sp, f, 3, nsteps, dt, w.omega, ev, ws)
        grads = []
        for _ in range(2):   # a second sweep finds the checkpoints as the first left them
            vbar, xbar = p.vel.clone(), torch.zeros_like(p.vel)
            g = torch.zeros((ctx.n_edge, 2), dtype=torch.float64, device="cuda")
            ctx.backward(n, sp, f, 3, nsteps, dt, w.omega, ev, ws, vbar, xbar, g)
            grads.append((vbar, xbar, g))
        for a, b in zip(*grads):
            assert torch.allclose(a, b, rtol=0, atol=1e-13 * a.abs().max().item())
        out.append((p, grads[0]))
    q = p0.clone()
    dG = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    for j in range(nsteps):
        ctx.gather_push_deposit(q, sp, f, 3 + j, dt, w.omega, dG)
    ctx.check()
    for p, _ in out:
        same_state(p.to_numpy(), q.to_numpy())
    print(f"[reverse] moved to another tet: {(q.tet != p0.tet).double().mean().item():.3f}", flush=True)
    for a, b in zip(out[0][1], out[1][1]):
        assert torch.allclose(a, b, rtol=0, atol=1e-12 * b.abs().max().item())
    ctx.close()


# one launch's most steps and one more, of few particles and of more than few
@pytest.mark.parametrize("n,nsteps", [(65, 32), (65, 65), (32768, 17), (32769, 17)])
def test_steps_per_launch(E, torch_cuda, n, nsteps):
    test_multi_equals_single_steps(E, torch_cuda, n, False, nsteps, 300.0, False, 0)


# 1 and 3 reverse launches per sweep; more particles than the first parts of the leavers' queue take
@pytest.mark.parametrize("n,nsteps,every", [(40_001, 5, 5), (40_001, 11, 11), (40_001, 4, 5)])
def test_reverse_sweeps_in_a_row_start_from_empty_queues(E, torch_cuda, n, nsteps, every):
    """Sweeps with an odd number of launches on one context, one after the
    other, against a context that has made none: the same derivatives to the
    rounding of the sums (1e-13 of the largest, as above)."""
    torch = torch_cuda

    def sweeps(many):
        w, ctx, f, sp, p = problem(E, torch, n, 0, True)
        p.vel *= 30.0
        start = p.tet.clone()
        ws = torch.empty(ctx.adjoint_workspace_bytes(n, nsteps, every), dtype=torch.uint8, device="cuda")
        ctx.forward_checkpointed(p, sp, f, 3, nsteps, 1e-9, w.omega, every, ws)
        assert (p.tet != start).double().mean().item() > 0.01
        for _ in range(many):
            vbar, xbar = p.vel.clone(), torch.zeros_like(p.vel)
            g = torch.zeros((ctx.n_edge, 2), dtype=torch.float64, device="cuda")
            ctx.backward(n, sp, f, 3, nsteps, 1e-9, w.omega, every, ws, vbar, xbar, g)
        ctx.check()
        ctx.close()
        return vbar, xbar, g
    for got, want in zip(sweeps(3), sweeps(1)):
        assert torch.allclose(got, want, rtol=0, atol=1e-13 * want.abs().max().item())


@pytest.mark.parametrize("downshifted", [False, True])
def test_timed_call_without_room_for_its_events_changes_nothing(E, torch_cuda, downshifted):
    """All but one of the 512 event sets taken: a timed call of two launches is
    refused before the first of them, and the call after it finds nothing
    queued or half deposited."""
    torch = torch_cuda
    n, nsteps, dt_scale = 1000, 33, 100.0
    w, ctx, f, sp, p = problem(E, torch, n, 0, False)
    dt, timed = w.dt * dt_scale, E.STEP_XCD_REMAP | E.STEP_TIMING
    g = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    q = p.clone()
    for j in range(511):
        ctx.gather_push_deposit(q, sp, f, j, w.dt, w.omega, g, flags=timed)
    hist = ctx.ds_history(p) if downshifted else None

    def call(ctx, p, hist, g, flags):
        if downshifted:
            ctx.ds_steps(p, hist, sp, f, 5, nsteps, 0, 1e-2 * dt, w.omega, g, flags=flags)
        else:
            ctx.run_steps(p, sp, f, 5, nsteps, dt, w.omega, g, flags=flags)
    g.zero_()
    before = p.clone()
    with pytest.raises(E.EtpicError) as ei:
        call(ctx, p, hist, g, timed)
    assert ei.value.code == E.EINVAL
    same_state(p.to_numpy(), before.to_numpy())
    assert torch.count_nonzero(g).item() == 0
    assert ctx.kernel_time()[1] == 511
    call(ctx, p, hist, g, timed)
    ctx.check()
    _, fresh, _, _, q = problem(E, torch, n, 0, False)
    g2 = torch.zeros_like(g)
    call(fresh, q, fresh.ds_history(q) if downshifted else None, g2, E.STEP_XCD_REMAP)
    fresh.check()
    same_state(p.to_numpy(), q.to_numpy())
    assert torch.allclose(g, g2, rtol=0, atol=1e-13 * g2.abs().max().item())
    ctx.close()
    fresh.close()


# meshes below and above 65,536 tets, few and more than few particles
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("side,n,nsteps", [(5, 65, 2), (5, 40_001, 2), (5, 1000, 3), (23, 1000, 3), (23, 32_769, 3),
                                           (23, 70_001, 2), (5, 1000, 4)])
def test_short_coarse_calls_equal_single_steps(E, torch_cuda, side, n, nsteps, precision):
    """Two and three fine steps with three different snapshots against the same
    call with its slices forced to one, which takes one step per launch."""
    torch = torch_cuda
    xyz, tv = synth.kuhn_mesh((side, side, side), (1.0, 1.0, 1.0), 0.1, np.random.default_rng(4))
    ctx = E.Context(0)
    ctx.upload_mesh(xyz, tv)
    g = torch.Generator(device="cuda").manual_seed(8)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float64, device="cuda", generator=g)
    b_dc, omega = 1e-4 * rnd(ctx.n_face), 2 * np.pi * 1e9
    snaps = [E.Fields(10.0 * rnd(ctx.n_edge, 2), 1e-5 * rnd(ctx.n_face, 2), None, b_dc) for _ in range(3)]
    lam = torch.rand(3, n, dtype=torch.float64, device="cuda", generator=g).sort(dim=0)[0].cpu().numpy()
    lam = np.stack([lam[0], lam[1] - lam[0], lam[2] - lam[1]], 1)
    tet = np.sort(np.random.default_rng(9).integers(tv.shape[0], size=n)).astype(np.int32)
    p1 = E.Particles.from_numpy(tet, lam, 1e6 * rnd(n, 3).cpu().numpy(), np.arange(n), precision=precision)
    p2 = p1.clone()
    sp = E.Species(synth.Q_E, synth.M_E, 1.0)
    g1 = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
    g2 = torch.zeros_like(g1)
    rho1 = torch.zeros(ctx.n_vert, dtype=torch.float64, device="cuda")
    rho2 = torch.zeros_like(rho1)
    dtc = nsteps * 0.05 / side / 1e6
    for _ in range(2):
        ctx.coarse_step(p1, sp, snaps, 3 * dtc, dtc, nsteps, omega, g1, rho=rho1)
        ctx.coarse_step(p2, sp, snaps, 3 * dtc, dtc, nsteps, omega, g2, rho=rho2, flags=E.STEP_XCD_REMAP | E.STEP_SLICES_1)
    ctx.check()
    assert (p1.tet.cpu().numpy() != tet).mean() > 0.01
    same_state(p1.to_numpy(), p2.to_numpy())
    assert torch.allclose(g1, g2, rtol=0, atol=1e-13 * g2.abs().max().item())
    assert torch.allclose(rho1, rho2, rtol=0, atol=1e-13 * rho2.abs().max().item())
    ctx.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n,ordered,nsteps", [(65, False, 7), (40_001, True, 10)])
def test_coarse_step_without_wide_rows(E, torch_cuda, n, ordered, nsteps, precision):
    """A context to which no wide rows were given takes two steps per launch:
    the results of one that has them."""
    torch = torch_cuda
    out = []
    for bound in (True, False):
        w, ctx, f, sp, p = problem(E, torch, n, precision, ordered)
        snaps = [E.Fields.from_numpy(e, b, None, w.b_dc) for e, b in synth.envelope_snapshots(w, seed=3)]
        if not bound:
            ctx._bind_wide_rows = lambda stream: None
        g = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
        dtc = nsteps * 300.0 * w.dt
        for k in range(2):
            ctx.coarse_step(p, sp, snaps, (3 + k) * dtc, dtc, nsteps, w.omega, g)
        ctx.check()
        assert (ctx._ds_rows is not None) == bound
        out.append((p.to_numpy(), g))
        ctx.close()
    same_state(out[0][0], out[1][0])
    assert torch.allclose(out[0][1], out[1][1], rtol=0, atol=1e-13 * out[0][1].abs().max().item())


# 32768 and 32769: 16 and 64 particles to a wavefront; 749 and 750 on 750 tets: the
# currents of one step straight to the edges and by the tets' slots
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,calls,edc", [(1, 3, False), (749, 6, True), (750, 6, False), (32768, 5, False), (32769, 5, True)])
def test_one_step_downshifted_calls_equal_one_call(E, torch_cuda, n, calls, edc, precision):
    """As test_downshifted_launch_split_changes_nothing."""
    test_downshifted_launch_split_changes_nothing(E, torch_cuda, n, n > 1000, calls, 100.0 if n > 1000 else 1.0, edc, False,
                                                  precision)


@pytest.mark.parametrize("precision", [0, 2])
@pytest.mark.parametrize("sorting", [False, True])
def test_more_leavers_than_the_queue_holds(E, torch_cuda, sorting, precision):
    """Twelve million particles, most of which leave their tet in the first
    step: each of the queue's 64 parts (131,072 entries) runs over, so leavers
    go by their slice or, in a sorting launch, by a scan of all particles; two
    steps in one launch against one step per launch.  Identical particles; an
    edge sums about 1e5 terms in another order (3e-14 of them by chance): 1e-12."""
    torch = torch_cuda
    n, side = 12_000_000, 5
    xyz, tv = synth.kuhn_mesh((side, side, side), (1.0, 1.0, 1.0), 0.1, np.random.default_rng(4))
    ctx = E.Context(0)
    ctx.upload_mesh(xyz, tv)
    gen = torch.Generator(device="cuda").manual_seed(8)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    f = E.Fields(0.1 * rnd(ctx.n_edge, 2), 1e-5 * rnd(ctx.n_face, 2), None, 1e-4 * rnd(ctx.n_face))
    sp = E.Species(synth.Q_E, synth.M_E, 1.0)
    lam = torch.rand(3, n, dtype=torch.float64, device="cuda", generator=gen).sort(dim=0)[0]
    lam = torch.stack([lam[0], lam[1] - lam[0], lam[2] - lam[1]])
    v = rnd(3, n)
    v *= 1e6 / v.norm(dim=0)
    tet = torch.randint(tv.shape[0], (n,), device="cuda", generator=gen, dtype=torch.int32).sort()[0]
    if precision == 2:
        u = (lam * (1.0 - 2e-9) * 4294967296.0).long()
        lam, v = torch.where(u >= 1 << 31, u - (1 << 32), u).int(), v.float()
    src = E.Particles(lam.contiguous(), v.contiguous(), tet, torch.arange(n, device="cuda"))
    dt, omega, out = 0.3 / 1e6, 2 * np.pi * 1e9, []
    for flags in (E.STEP_XCD_REMAP, E.STEP_XCD_REMAP | E.STEP_SLICES_1):
        g = torch.zeros(ctx.n_edge, dtype=torch.float64, device="cuda")
        p = src.empty_like() if sorting else src.clone()
        if sorting:
            ctx.sort_run_steps(src, p, sp, f, 0, 2, dt, omega, g, flags=flags)
        else:
            ctx.run_steps(p, sp, f, 0, 2, dt, omega, g, flags=flags)
        ctx.check()
        o = p.ids.argsort()
        out.append((p.tet[o], p.lam[:, o], p.vel[:, o], g))
    moved = (out[0][0] != tet).double().mean().item()
    print(f"[multi] moved to another tet: {moved:.3f}", flush=True)
    assert moved * n > 64 * 131072
    for a, b in zip(out[0][:3], out[1][:3]):
        assert torch.equal(a, b)
    assert torch.allclose(out[0][3], out[1][3], rtol=0, atol=1e-12 * out[1][3].abs().max().item())
    ctx.close()
