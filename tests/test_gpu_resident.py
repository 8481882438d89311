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


# ---- several streams and threads -------------------------------------------------
# grid, precision, tolerance: solves that share the device, and ones that need
# it to themselves
KINDS = [(32, 0, 1e-10), (32, 1, 1e-6), (48, 0, 1e-9), (64, 1, 1e-7), (100, 0, 1e-8)]


def alone_fields(maze, kind, seed, steps):
    """Fields of a session stepped with nothing else on the device."""
    s, x = make(maze, *kind, seed)
    out = []
    for k in range(steps):
        assert x.step(dev(s.pos + (k + 1) * s.vel))["status"] == 0
        out.append(x.grid(maze.GRID_PHI).clone())
    x.close()
    torch.cuda.synchronize()
    return out


def on_stream(maze, kind, seed, stream):
    with torch.cuda.stream(stream):
        return make(maze, *kind, seed, stream=stream.cuda_stream)


def kept_resident(maze, *sessions):
    for x in sessions:
        got = maze.maze_resident_solves(x.handle)
        assert got["resident"] and got["given_up"] == 0, got


def test_threads_with_streams_of_their_own(maze):
    """A session a thread, each on its own stream: every step's field is the
    one it gets alone, and no solve gives up."""
    import threading
    steps = 40
    print(f"case: threads {KINDS}", flush=True)
    want = [alone_fields(maze, k, 80 + i, steps) for i, k in enumerate(KINDS)]
    made = [on_stream(maze, k, 80 + i, torch.cuda.Stream()) for i, k in enumerate(KINDS)]
    pos = [[dev(s.pos + (k + 1) * s.vel) for k in range(steps)] for s, _ in made]
    torch.cuda.synchronize()
    got = [[] for _ in KINDS]
    failed = []

    def work(i):
        try:
            x = made[i][1]
            for k in range(steps):
                assert x.step(pos[i][k])["status"] == 0
                got[i].append(x.grid(maze.GRID_PHI))
        except BaseException as e:  # noqa: BLE001
            failed.append((i, e))
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(KINDS))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    kept_resident(maze, *(x for _, x in made))
    for i in range(len(KINDS)):
        for k in range(steps):
            assert torch.equal(got[i][k], want[i][k]), (KINDS[i], k)
    for _, x in made:
        x.close()


def test_continuous_batches_beside_steps_on_other_streams(maze):
    """Two continuous batches, whose resident solves nobody waits for, and steps
    of other sessions, on three streams: each result is the one alone."""
    print(f"case: two batches and steps on three streams {KINDS}", flush=True)
    want = [alone_fields(maze, k, 90 + i, 3) for i, k in enumerate(KINDS)]
    s1, s2, s3 = (torch.cuda.Stream() for _ in range(3))
    groups = [[on_stream(maze, k, 90 + i, st) for i, k in enumerate(KINDS)] for st in (s1, s2, s3)]
    batches = [maze.Batch(max_sessions=8, stream=s1.cuda_stream),
               maze.Batch(max_sessions=8, stream=s2.cuda_stream)]
    for k in range(3):
        left = [len(KINDS), len(KINDS)]
        p = [dev(s.pos + (k + 1) * s.vel) for s, _ in groups[0]]
        torch.cuda.synchronize()
        for b, g in zip(batches, groups):
            for i, (_, x) in enumerate(g):
                b.add(x.handle, p[i], tag=i)
        own = list(enumerate(groups[2]))
        for _ in range(100000):
            for j, b in enumerate(batches):
                if left[j]:
                    b.advance()
                    for tag, st in b.take():
                        assert st["status"] == 0
                        left[j] -= 1
            if own:
                i, (_, x) = own.pop()
                assert x.step(p[i])["status"] == 0
            if not any(left) and not own:
                break
        assert not any(left) and not own
        torch.cuda.synchronize()
        for g in groups:
            for i, (_, x) in enumerate(g):
                assert torch.equal(x.grid(maze.GRID_PHI), want[i][k]), (KINDS[i], k)
    for g in groups:
        kept_resident(maze, *(x for _, x in g))
        for _, x in g:
            x.close()
    for b in batches:
        b.close()


@pytest.mark.parametrize("kind", [(32, 0, 1e-9), (100, 0, 1e-6)])
def test_a_step_is_not_held_by_another_streams_queue(maze, kind):
    """A thread whose stream still has a second of the caller's work before its
    step: steps on other streams meanwhile take as long as ever."""
    import threading
    import time
    a = torch.cuda.Stream()
    with torch.cuda.stream(a):  # cycles of half a second, from a short sleep
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda._sleep(1000)
        e0.record()
        torch.cuda._sleep(10000000)
        e1.record()
    a.synchronize()
    half = int(10000000 * 500.0 / e0.elapsed_time(e1))
    one = torch.ones(1, device="cuda")
    b = None
    for _ in range(8):  # a stream that does not share a's hardware queue
        c = torch.cuda.Stream()
        with torch.cuda.stream(a):
            torch.cuda._sleep(half // 5)
        t0 = time.perf_counter()
        with torch.cuda.stream(c):
            one.add_(1)
        c.synchronize()
        if time.perf_counter() - t0 < 0.05:
            b = c
        a.synchronize()
        if b is not None:
            break
    if b is None:
        pytest.skip("no stream beside the first one")
    print(f"case: step beside another stream's queue {kind}", flush=True)
    sa, xa = on_stream(maze, kind, 70, a)
    sb, xb = on_stream(maze, kind, 71, b)
    pa, pb = dev(sa.pos + sa.vel), dev(sb.pos + sb.vel)
    torch.cuda.synchronize()
    for x, p in ((xa, pa), (xb, pb), (xa, pa), (xb, pb)):
        x.step(p)
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        torch.cuda._sleep(2 * half)
    t = threading.Thread(target=lambda: xa.step(pa))
    t.start()
    time.sleep(0.1)
    t0 = time.perf_counter()
    for _ in range(3):
        xb.step(pb)
    took = time.perf_counter() - t0
    waiting = t.is_alive()
    t.join()
    torch.cuda.synchronize()
    assert waiting and took < 0.4, (waiting, took)
    kept_resident(maze, xa, xb)
    xa.close()
    xb.close()


# exchange partly in memory of its own (20, 32, 44) and all in that of launched
# solves' vectors
@pytest.mark.parametrize("N,prec,tol", [(20, 0, 1e-10), (32, 1, 1e-7), (40, 0, 1e-9),
                                        (44, 0, 1e-9),
                                        (64, 1, 1e-7), (96, 0, 1e-9), (128, 1, 1e-6)])
@pytest.mark.parametrize("sstep", [False, True])
def test_forms_follow_each_other(maze, monkeypatch, N, prec, tol, sstep):
    """Launched solves (timed steps, batches above the fill level, direct solves
    among them) leave their vectors where the next resident solve keeps its
    exchange: the forms may follow each other in any order."""
    print(f"case: resident and launched solves in turn, N {N} precision {prec}", flush=True)
    flags = maze.MAZE_FLAG_SSTEP if sstep else 0
    s, a = make(maze, N, prec, tol, 40 + N, flags=flags)
    _, other = make(maze, N, prec, tol, 41 + N, flags=flags)
    monkeypatch.setenv("MAZE_PERSIST", "0")
    _, b = make(maze, N, prec, tol, 40 + N, flags=flags)
    monkeypatch.delenv("MAZE_PERSIST")
    bound = field_bound(s, a, N, tol, maze)
    plan = ["resident", "timed", "resident", "resident", "batch", "resident", "solve", "timed",
            "solve", "resident"]
    for k, form in enumerate(plan):
        p = dev(s.pos + (k + 1) * s.vel)
        before = maze.maze_resident_solves(a.handle)["solves"]
        if form == "timed":
            maze.maze_profile_enable(a.handle, True)
        if form == "solve":
            fa, fb = a.solve(p)["field"], b.solve(p)["field"]
            assert torch.linalg.norm(fa - fb).item() <= bound, (k, form)
        elif form == "batch":
            monkeypatch.setenv("MAZE_BATCH_MODE", "throughput")
            assert maze.maze_step_batch([a.handle, other.handle], [p, p])[0] == 0
            monkeypatch.delenv("MAZE_BATCH_MODE")
        else:
            assert a.step(p)["status"] == 0
        if form != "solve":
            assert b.step(p)["status"] == 0
        maze.maze_profile_enable(a.handle, False)
        ran = maze.maze_resident_solves(a.handle)["solves"] - before
        assert (ran > 0) == (form in ("resident", "solve")), (k, form, ran)
        d = torch.linalg.norm(a.grid(maze.GRID_PHI) - b.grid(maze.GRID_PHI)).item()
        assert d <= (k + 1) * bound, (k, form, d)
    kept_resident(maze, a)
    for x in (a, b, other):
        x.close()


def test_resident_again_after_a_solve_that_gave_up(maze, monkeypatch):
    """A solve that gave up costs the session its next 64 resident solves, the
    second one 128; in between they are resident again, from a clean exchange."""
    N, tol = 20, 1e-9
    print("case: resident again after a solve given up", flush=True)
    s, x = make(maze, N, 0, tol, 15)
    _, y = make(maze, N, 0, tol, 16)
    monkeypatch.setenv("MAZE_PERSIST", "0")
    _, ref = make(maze, N, 0, tol, 15)
    monkeypatch.delenv("MAZE_PERSIST")
    p = [dev(s.pos + s.vel * math.sin(0.3 * (k + 1))) for k in range(7)]
    bound = field_bound(s, x, N, tol, maze)
    k, rests = 0, (64, 128)
    for lost, rest in enumerate(rests, 1):
        monkeypatch.setenv("MAZE_PERSIST_SPIN", "0")
        assert x.step(p[k % 7])["status"] == 0
        monkeypatch.delenv("MAZE_PERSIST_SPIN")
        ref.step(p[k % 7])
        k += 1
        done = maze.maze_resident_solves(x.handle)["solves"]
        # the step's own repetition is the first of them; a batch's members
        # that are launched and those that are not keep their places
        for i in range(rest - 1):
            got = maze.maze_resident_solves(x.handle)
            assert got == dict(resident=False, solves=done, given_up=lost), (lost, i)
            if i == rest - 2:
                assert maze.maze_step_batch([y.handle, x.handle], [p[k % 7], p[k % 7]])[0] == 0
            else:
                assert x.step(p[k % 7])["status"] == 0
            ref.step(p[k % 7])
            k += 1
        assert maze.maze_resident_solves(x.handle)["resident"]
        for i in range(3):
            assert x.step(p[k % 7])["status"] == 0
            ref.step(p[k % 7])
            k += 1
        got = maze.maze_resident_solves(x.handle)
        assert got == dict(resident=True, solves=done + 3, given_up=lost)
        # each step of either leaves its residual, and a step's error reaches
        # the next one twice over at most: the last ones bound the rest
        d = torch.linalg.norm(x.grid(maze.GRID_PHI) - ref.grid(maze.GRID_PHI)).item()
        assert d <= k * bound, (k, d)
    kept = maze.maze_resident_solves(y.handle)
    assert kept["given_up"] == 0
    for z in (x, y, ref):
        z.close()


def test_stream_with_some_of_the_compute_units(maze):
    """On a stream restricted to a part of the device, a solve's workgroups might
    not all be resident: its sessions are launched ones from the start."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    words = (cus + 31) // 32
    mask = (ctypes.c_uint32 * words)(*[0x0000FFFF] * words)
    st = ctypes.c_void_p()
    if hip.hipExtStreamCreateWithCUMask(ctypes.byref(st), words, mask) != 0:
        pytest.skip("no CU mask on this device")
    print("case: a stream with half of the compute units", flush=True)
    s, x = make(maze, 64, 0, 1e-9, 17, stream=st.value)
    _, y = make(maze, 64, 0, 1e-9, 17)
    p = dev(s.pos + s.vel)
    torch.cuda.synchronize()
    assert maze.maze_resident_solves(y.handle)["resident"]
    got = maze.maze_resident_solves(x.handle)
    assert got == dict(resident=False, solves=0, given_up=0)
    assert x.step(p)["status"] == 0 and y.step(p)["status"] == 0
    torch.cuda.synchronize()
    d = torch.linalg.norm(x.grid(maze.GRID_PHI) - y.grid(maze.GRID_PHI)).item()
    assert d <= field_bound(s, y, 64, 1e-9, maze)
    x.close()
    y.close()
    hip.hipStreamDestroy(st)


def test_steps_get_their_turn_beside_busy_batches(maze):
    """Two threads that keep continuous batches of large solves going, each
    queueing its next solve behind the other's: a session on a stream of its own
    still gets its turn."""
    import threading
    import time
    kind = (96, 0, 1e-8)
    print(f"case: steps beside busy batches {kind}", flush=True)
    want = alone_fields(maze, kind, 60, 4)
    stop, failed = threading.Event(), []

    def busy(seed):
        try:
            st = torch.cuda.Stream()
            made = [on_stream(maze, kind, seed + i, st) for i in range(2)]
            b = maze.Batch(max_sessions=4, stream=st.cuda_stream)
            pos = [[dev(s.pos + f * s.vel) for f in (1.0, 2.0)] for s, _ in made]
            torch.cuda.synchronize()
            ready.wait()
            k, flying = [0, 0], [False, False]
            while not stop.is_set() or any(flying):
                for i, (_, x) in enumerate(made):
                    if not flying[i] and not stop.is_set():
                        b.add(x.handle, pos[i][k[i] % 2], tag=i)
                        k[i] += 1
                        flying[i] = True
                b.advance()
                for tag, res in b.take():
                    assert res["status"] == 0
                    flying[tag] = False
            kept_resident(maze, *(x for _, x in made))
            b.close()
            for _, x in made:
                x.close()
        except BaseException as e:  # noqa: BLE001
            failed.append(e)
            stop.set()
    ready = threading.Barrier(3)
    threads = [threading.Thread(target=busy, args=(20 * t,)) for t in (1, 2)]
    for t in threads:
        t.start()
    s, x = on_stream(maze, kind, 60, torch.cuda.Stream())
    pos = [dev(s.pos + (k + 1) * s.vel) for k in range(4)]
    torch.cuda.synchronize()
    ready.wait()
    time.sleep(0.05)
    t0 = time.perf_counter()
    for k in range(4):
        assert x.step(pos[k])["status"] == 0
        assert torch.equal(x.grid(maze.GRID_PHI), want[k]), k
    took = time.perf_counter() - t0
    stop.set()
    for t in threads:
        t.join()
    assert not failed, failed
    assert took < 1.0, took  # four of 1.4 ms alone, each behind some of theirs
    kept_resident(maze, x)
    x.close()
