"""bench.py's timed steps are those a caller gets."""
import os
import sys

import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2505_20418_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("persist,form", [(None, "resident"), ("0", "launched")])
def test_sampling_does_not_change_the_timed_form(monkeypatch, persist, form):
    """The sampling of the launched kernels' times switches a session of resident
    solves to those, so it stays out of the steps that are timed."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import bench
    from paper_2505_20418_amd import maze
    if persist is not None:
        monkeypatch.setenv("MAZE_PERSIST", persist)
    timed, steps = [], 40
    read = maze.maze_md_step

    def step(handle, md, want_stats=True):
        before = maze.maze_resident_solves(handle)["solves"]
        out = read(handle, md, want_stats)
        timed.append(maze.maze_resident_solves(handle)["solves"] - before)
        return out
    monkeypatch.setattr(maze, "maze_md_step", step)
    print(f"case: timed steps of {form} solves", flush=True)
    r = bench.run_md(inputs.molten_nacl(2, seed=3), 1e-9, maze.MAZE_FP64, steps, 2)
    assert r["form"] == form
    assert all((n > 0) == (form == "resident") for n in timed[:2 + steps])
    # the kernels were sampled all the same, in every step's solve
    assert r["prof"]["fp64_sweep"][0] >= steps and r["prof"]["fp64_iters"] > 10 * steps
    assert len(r["lat_ms"]) == steps and r["steps_per_s"] > 0
