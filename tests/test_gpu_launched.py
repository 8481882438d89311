"""The launched solves (fused sweeps, two-iteration kernels, batched launch
tables, captured poll groups) on the grids that resident solves take over: the
tests of those kernels, run again with MAZE_PERSIST=0. They still serve larger
grids, batches above the fill level, timed sessions and repeated solves."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2505_20418_amd import inputs  # noqa: E402
from test_gpu_batch import (  # noqa: E402,F401
    test_batch_is_bitwise_alone, test_batch_member_matches_oracle,
    test_batch_rejected_member_is_unchanged, test_throughput_mode_within_tolerance_of_alone)
from test_gpu_continuous import (  # noqa: E402,F401
    test_md_steps_in_batch_bitwise_alone, test_rejected_step_leaves_session_unchanged,
    test_steps_join_running_batch_bitwise_alone, test_throughput_shapes_meet_tolerance)
from test_gpu_graph import (  # noqa: E402,F401
    gpu, test_batch_graph_groups_bitwise, test_graph_chunks_bitwise_equal,
    test_graph_chunks_follow_the_solution_vector)
from test_gpu_parity import (  # noqa: E402,F401
    test_absmax_residual_norm, test_bitwise_determinism_and_checkpoint,
    test_direct_solve_guesses, test_errors_leave_state_unchanged, test_init_and_steps_match_oracle,
    test_lockstep_cg_iterates, test_md_matches_oracle_md, test_mixed_precision_error_vs_fp64_oracle,
    test_ragged_grids)
from test_gpu_sstep import (  # noqa: E402,F401
    maze, test_first_pass_on_device_matches_host_decided, test_sstep_absmax_residual_norm,
    test_sstep_batch_is_bitwise_alone, test_sstep_batch_throughput_mode,
    test_sstep_direct_solve_guesses, test_sstep_fixed_iteration_count,
    test_sstep_graph_chunks_bitwise, test_sstep_mixed_precision, test_sstep_ragged_grids,
    test_sstep_steps_match_oracle)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def launched(monkeypatch):
    monkeypatch.setenv("MAZE_PERSIST", "0")


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("N,prec", [(4, 0), (20, 1), (64, 0), (76, 1), (128, 0), (129, 0)])
def test_the_form_is_the_one_asked_for(maze, monkeypatch, N, prec):  # noqa: F811
    """Every session of this file solves by launched kernels; without the
    setting those of up to 128^3 are resident, in both CG forms."""
    print(f"case: form of N {N} precision {prec}", flush=True)
    s = inputs.molten_nacl(max(2, N // 16), seed=N)
    for flags in (0, maze.MAZE_FLAG_SSTEP):
        for setting in ("0", None):
            if setting is None:
                monkeypatch.delenv("MAZE_PERSIST")
            else:
                monkeypatch.setenv("MAZE_PERSIST", setting)
            x = maze.Session(dev(s.charges), dev(s.pos), s.box, s.box / N, tol=1e-6,
                             precision=prec, flags=flags)
            assert x.step(dev(s.pos + s.vel))["status"] == 0
            got = maze.maze_resident_solves(x.handle)
            resident = setting is None and N <= 128
            assert got["resident"] == resident and got["given_up"] == 0
            # the cold solve and the step, one inner solve each at least
            assert got["solves"] >= 2 if resident else got["solves"] == 0
            x.close()
