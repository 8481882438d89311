"""Resident solves: every CG iteration of a small grid in one launch.

The workgroups of a resident solve keep their brick of the grid in registers
and exchange boundary rows and sums among themselves. Its iterates are the
launched sweep's up to the rounding of the sums' order, so the field differs
from a launched session's by at most the two solves' residuals through the
inverse operator, (4 pi / h) 2 tol ||q|| / lambda_min with lambda_min =
2 (1 - cos(2 pi / N)) of the periodic 7-point M. A solve that gives up
waiting for its workgroups is repeated by launched kernels.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2505_20418_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def maze():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_20418_amd import maze as m
    m.lib()
    return m


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def make(maze, N, prec, tol, seed, **kw):
    s = inputs.molten_nacl(max(2, N // 16), seed=seed)
    s.grid_spacing = s.box / N
    return s, maze.Session(dev(s.charges), dev(s.pos), s.box, s.grid_spacing, tol=tol,
                           precision=prec, coulomb_k=inputs.COULOMB_K_EV_A, **kw)


def field_bound(s, g, N, tol, maze):
    qn = torch.linalg.norm(g.grid(maze.GRID_Q)).item()
    return ((4 * math.pi / (s.box / N)) * 2 * tol * qn
            / (2 * (1 - math.cos(2 * math.pi / N))))


# one workgroup (4), bricks of one shape and of two (9, 31, 33), threads past
# the brick's columns (50, 97), every thread count, the largest grids (112, 128)
@pytest.mark.parametrize("N", [4, 9, 31, 33, 50, 64, 97, 112, 128])
@pytest.mark.parametrize("prec,tol", [(0, 1e-10), (1, 1e-7)])
def test_resident_matches_launched(maze, monkeypatch, N, prec, tol):
    print(f"case: resident N {N} precision {prec}", flush=True)
    s, a = make(maze, N, prec, tol, 60 + N)
    monkeypatch.setenv("MAZE_PERSIST", "0")
    _, b = make(maze, N, prec, tol, 60 + N)
    monkeypatch.delenv("MAZE_PERSIST")
    for k in range(3):
        p = dev(s.pos + (k + 1) * s.vel)
        ra, rb = a.step(p, want_field=True), b.step(p, want_field=True)
        assert ra["status"] == rb["status"] == 0
        assert ra["stats"]["rel_residual"] <= tol
        assert abs(ra["stats"]["iters"] - rb["stats"]["iters"]) <= 2
        d = torch.linalg.norm(ra["field"] - rb["field"]).item()
        assert d <= field_bound(s, a, N, tol, maze), (k, d)
    sa, sb = a.solve(p), b.solve(p)
    assert abs(sa["stats"]["iters"] - sb["stats"]["iters"]) <= 2
    d = torch.linalg.norm(sa["field"] - sb["field"]).item()
    assert d <= field_bound(s, a, N, tol, maze)
    a.close()
    b.close()


@pytest.mark.parametrize("max_iter", [0, 1, 2, 13])
@pytest.mark.parametrize("norm", [0, 1])
def test_resident_stops_where_the_sweep_does(maze, monkeypatch, max_iter, norm):
    """The iteration cap and both norms: counts, codes and residuals."""
    tol = 1e-300 if max_iter < 13 else 1e-2
    kw = dict(max_iter=max_iter, residual_norm=norm)
    s, a = make(maze, 20, 0, tol, 7, **kw)
    monkeypatch.setenv("MAZE_PERSIST", "0")
    _, b = make(maze, 20, 0, tol, 7, **kw)
    monkeypatch.delenv("MAZE_PERSIST")
    p = dev(s.pos + s.vel)
    ra, rb = a.step(p, want_field=True), b.step(p, want_field=True)
    assert ra["status"] == rb["status"] and ra["stats"]["iters"] == rb["stats"]["iters"]
    # the same iterates after a fixed count: rounding only
    assert torch.linalg.norm(ra["field"] - rb["field"]) <= 1e-12 * torch.linalg.norm(rb["field"])
    a.close()
    b.close()


@pytest.mark.parametrize("prec,tol", [(0, 1e-10), (1, 1e-7)])
def test_solve_that_gives_up_is_repeated(maze, monkeypatch, prec, tol):
    """With no polls allowed, a workgroup leaves as soon as another's sums are
    not there yet: the solves are repeated by launched sweeps, alone, in a
    batch and in a continuous batch."""
    print(f"case: resident solve given up, precision {prec}", flush=True)
    N = 32
    monkeypatch.setenv("MAZE_PERSIST", "0")
    s, ref = make(maze, N, prec, tol, 11)
    monkeypatch.delenv("MAZE_PERSIST")
    _, alone = make(maze, N, prec, tol, 11)
    _, inbatch = make(maze, N, prec, tol, 11)
    _, other = make(maze, N, prec, tol, 11)
    _, flight = make(maze, N, prec, tol, 11)
    p = dev(s.pos + s.vel)
    want = ref.step(p, want_field=True)
    monkeypatch.setenv("MAZE_PERSIST_SPIN", "0")
    got = [alone.step(p, want_field=True)["field"]]
    rc, st = maze.maze_step_batch([inbatch.handle, other.handle], [p, p])
    assert rc == 0 and all(x["rel_residual"] <= tol for x in st)
    got += [inbatch.grid(maze.GRID_PHI), other.grid(maze.GRID_PHI)]
    batch = maze.Batch(max_sessions=4)
    batch.add(flight.handle, p, tag=1)
    done = []
    for _ in range(100000):
        batch.advance()
        done += batch.take()
        if done:
            break
    assert done[0][1]["status"] == 0 and done[0][1]["rel_residual"] <= tol
    got.append(flight.grid(maze.GRID_PHI))
    bound = field_bound(s, ref, N, tol, maze)
    for f in got:
        assert torch.linalg.norm(f - want["field"]).item() <= bound
    batch.close()
    for x in (ref, alone, inbatch, other, flight):
        x.close()


# one inner solve, several, none (a right-hand side within a loose tolerance), a
# step that may not converge, and FP64
@pytest.mark.parametrize("prec,tol,max_iter", [
    (0, 1e-10, 100000), (0, 1e-10, 5), (1, 1e-6, 100000), (1, 1e-12, 100000), (1, 0.5, 100000),
    (1, 1e-10, 9)])
@pytest.mark.parametrize("spin", [None, "0"])
def test_steps_queued_ahead_are_those_of_a_batch(maze, monkeypatch, prec, tol, max_iter, spin):
    """A step alone is queued whole before its solve has ended; in a batch the
    host waits for each stage. Both end in the same bits, where the solve ends
    as foreseen, where it needs more, and where it gives up and is repeated."""
    from paper_2505_20418_amd.md import MDRun, step_many
    print(f"case: queued ahead precision={prec} tol={tol} max_iter={max_iter} spin={spin}",
          flush=True)
    s = inputs.molten_nacl(2, seed=21)
    make_run = lambda: MDRun(s, tol=tol, precision=prec, max_iter=max_iter, gamma=0.01,
                             temperature=1000.0, seed=5)
    alone, a, b = make_run(), make_run(), make_run()
    if spin is not None:
        monkeypatch.setenv("MAZE_PERSIST_SPIN", spin)
    for _ in range(3):
        _, got = alone.step(want_stats=True)
        _, want = step_many([a, b])
        for x in (a, b):
            for name in ("pos", "vel", "f_es", "f_sr", "scalars"):
                assert torch.equal(getattr(alone, name), getattr(x, name)), name
        assert torch.equal(alone.session.grid(maze.GRID_PHI), a.session.grid(maze.GRID_PHI))
        assert got == want[0], (got, want[0])
    for x in (alone, a, b):
        x.close()


def test_queued_ahead_step_with_bad_positions_changes_nothing(maze):
    from paper_2505_20418_amd.md import MDRun
    s = inputs.molten_nacl(2, seed=22)
    run = MDRun(s, tol=1e-6, precision=1)
    run.step()
    keep = {k: getattr(run, k).clone() for k in ("f_es", "f_sr", "scalars")}
    phi, pos = run.session.grid(maze.GRID_PHI), run.pos.clone()
    vel = run.vel.clone()
    run.pos[3, 1] = float("nan")
    with pytest.raises(maze.MazeError):
        run.step()
    for k, v in keep.items():
        assert torch.equal(getattr(run, k), v), k
    assert torch.equal(run.session.grid(maze.GRID_PHI), phi)
    run.pos.copy_(pos)
    run.vel.copy_(vel)
    run.step()
    assert torch.isfinite(run.f_es).all() and torch.isfinite(run.scalars).all()
    run.close()


@pytest.mark.parametrize("prec,tol", [(0, 1e-10), (1, 1e-7)])
def test_given_up_solves_are_counted(maze, monkeypatch, prec, tol):
    """What a session reports of its solves, alone, in a batch and in a
    continuous batch: each was given up with no polls allowed, and none was
    with the polls there usually are."""
    N = 32
    for spin in (None, "0"):
        print(f"case: solves given up are counted, precision {prec}, spin {spin}", flush=True)
        monkeypatch.delenv("MAZE_PERSIST_SPIN", raising=False)
        s, alone = make(maze, N, prec, tol, 12)
        _, a = make(maze, N, prec, tol, 12)
        _, b = make(maze, N, prec, tol, 12)
        _, flight = make(maze, N, prec, tol, 12)
        p = dev(s.pos + s.vel)
        before = [maze.maze_resident_solves(x.handle) for x in (alone, a, b, flight)]
        assert all(x["resident"] and x["given_up"] == 0 for x in before)
        if spin is not None:
            monkeypatch.setenv("MAZE_PERSIST_SPIN", spin)
        assert alone.step(p)["status"] == 0
        assert maze.maze_step_batch([a.handle, b.handle], [p, p])[0] == 0
        batch = maze.Batch(max_sessions=4)
        batch.add(flight.handle, p, tag=1)
        done = []
        for _ in range(100000):
            batch.advance()
            done += batch.take()
            if done:
                break
        assert done[0][1]["status"] == 0
        for x, old in zip((alone, a, b, flight), before):
            now = maze.maze_resident_solves(x.handle)
            if spin is None:
                assert now["given_up"] == 0 and now["solves"] > old["solves"]
            else:
                assert now["given_up"] == 1 and now["solves"] == old["solves"]
                assert not now["resident"]
        batch.close()
        for x in (alone, a, b, flight):
            x.close()
