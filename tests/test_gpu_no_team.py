"""Solves whose team of resident workgroups does not come together (other
programs' work holds the CUs; here the wait for it is set to 0, so the
launch leaves at once): the launch-per-kernel solver and the one-workgroup
batch kernel take them from the x the caller gave, and do everything that the
solver's and the batch's own tests ask for."""
import time

import numpy as np
import pytest

import oracle
import paper_2409_15468_amd as cb
import synth
from tests import test_gpu_batch as batch
from tests import test_gpu_server as server
from tests import test_gpu_solve as solve

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_teams():
    cb.lib().cb_internal_team_wait(0, 0)
    yield
    cb.lib().cb_internal_team_wait(-1, 0)


@pytest.mark.parametrize("fmt", solve.FORMATS)
def test_solve_formats(fmt):
    solve.test_plain_config_all_formats(fmt)


@pytest.mark.parametrize("l", [8, 12, 18, 24, 28])
def test_solve_generic_widths(l):
    solve.test_generic_width_solves(l)


@pytest.mark.parametrize("l", [16, 21])
def test_solve_generic_codec_is_the_specialised_one(l):
    solve.test_generic_codec_solve_is_the_specialised_solve(l)


@pytest.mark.parametrize("fmt", ["frsz2b64_16", "frsz2b64_32", "frsz2b64_21"])
def test_solve_block64(fmt):
    solve.test_block64_solves(fmt)


@pytest.mark.parametrize("fmt", ["float64", "frsz2_21"])
@pytest.mark.parametrize("N,m", [(3, 4), (5, 1), (23, 7), (47, 100)])
def test_solve_ragged(fmt, N, m):
    solve.test_small_ragged_and_restart_lengths(fmt, N, m)


def test_solve_edges_caps_and_nonfinite_input():
    solve.test_edge_cases()


def test_solve_literal_breakdown():
    solve.test_literal_breakdown_option()


@pytest.mark.parametrize("fmt,m", [("frsz2_16", 40), ("frsz2_32", 40)])
def test_refinement(fmt, m):
    s = synth.plain_2d(N=48, seed=3)
    ref = oracle.ir_solve(s.A, s.b, m, 1e-4, 1e-12, fmt)
    A = cb.DeviceCSR.from_host(s.A.row_ptr, s.A.col, s.A.val)
    x = torch.zeros(s.A.n, dtype=torch.float64, device="cuda")
    res = cb.cbgmres_ir_solve(A, torch.from_numpy(s.b).cuda(), x, m, 1e-4, 1e-12, fmt)
    assert res["converged"] and solve.host_rrn(s.A, s.b, x.cpu().numpy()) <= 1e-12 + 1e-14
    assert res["restarts"] == ref.outer and solve.within_2pct(res["iterations"], ref.iterations)


@pytest.mark.parametrize("launches", [1, 2])
def test_solve_goes_on_where_the_teams_ended(launches, m=1):
    """With a history and m = 1 a launch of a team runs 224 steps (as many as
    its workspace has entries for).  After `launches` of them no more team forms:
    the rest of the solve counts on -- iterations, restarts, history, both caps."""
    A = synth.convection_diffusion(50, 2, (20.0, 0.0))
    b = synth.rhs_from_solution(A, np.random.default_rng(3).uniform(-1, 1, A.n))
    for caps in ({"max_iters": 700}, {"max_cycles": 640 // m}):
        cb.lib().cb_internal_team_wait(0, launches)
        res, x, hist = solve.gpu_solve(A, b, m, 1e-12, "float64", history_cap=5000, **caps)
        ref = oracle.gmres(A, b, m, 1e-12, "float64", hist_cap=5000, **caps)
        assert ref.iterations > 2 * 224 and not ref.converged
        assert res["status"] == cb.CB_ERR_NOT_CONVERGED
        assert res["iterations"] == ref.iterations == hist.size and res["restarts"] == ref.restarts
        assert abs(res["reorths"] - ref.reorths) <= max(2, 0.02 * ref.reorths)
        np.testing.assert_allclose(hist, ref.history, rtol=1e-5)
        assert np.linalg.norm(x - ref.x) <= 1e-8 * np.linalg.norm(ref.x)


def test_solve_converges_where_the_teams_ended():
    """The same with m = 3 (74 cycles a launch), to convergence."""
    cb.lib().cb_internal_team_wait(0, 1)
    A = synth.convection_diffusion(50, 2, (20.0, 0.0))
    b = synth.rhs_from_solution(A, np.random.default_rng(3).uniform(-1, 1, A.n))
    ref = oracle.gmres(A, b, 3, 1e-10, "float64", hist_cap=5000)
    assert ref.converged and ref.iterations > 300
    res, x, hist = solve.gpu_solve(A, b, 3, 1e-10, "float64", history_cap=5000)
    assert res["converged"] and solve.host_rrn(A, b, x) <= 1e-10 * (1 + 1e-6)
    assert solve.within_2pct(res["iterations"], ref.iterations) and hist.size == res["iterations"]


def test_batch_formats():
    batch.test_plain_config_all_formats_one_batch()


@pytest.mark.parametrize("fmt", batch.FORMATS)
def test_batch_columns(fmt):
    batch.test_first_cycle_columns_follow_oracle(fmt)


def test_batch_alone_equals_mixed():
    batch.test_alone_equals_mixed()


def test_batch_many_systems_per_workgroup():
    batch.test_many_systems_per_workgroup()


@pytest.mark.parametrize("fmt", ["float64", "frsz2_21"])
@pytest.mark.parametrize("n,m", [(1, 3), (33, 4), (100, 1), (1000, 25), (5000, 104)])
def test_batch_ragged(fmt, n, m):
    batch.test_ragged_sizes_and_restarts(fmt, n, m)


def test_batch_edges():
    batch.test_edge_cases()
    batch.test_literal_breakdown_option()


def test_served_requests():
    server.test_alone_equals_mixed_and_meets_tolerance()


def test_served_result_is_the_batch_s():
    """The served x is, bit for bit, that of a batch without teams."""
    A = synth.convection_diffusion(45, 2, (20.0, 0.0))
    b = synth.rhs_from_solution(A, np.random.default_rng(8).uniform(-1, 1, A.n))
    x0 = np.random.default_rng(9).uniform(-1, 1, A.n)
    res, xs, _ = batch.batch([(A, b, 30, 1e-9, "frsz2_21", x0)])
    srv = cb.Server(1 << 30, 0, lanes=1)
    t = srv.submit(A.row_ptr, A.col, A.val, b, 30, 1e-9, "frsz2_21", x0=x0)
    got, t0 = None, time.time()
    while got is None and time.time() - t0 < 20:
        time.sleep(0.001)
        got = srv.poll(t, A.n)
    srv.close()
    assert got is not None and np.array_equal(got[0], xs[0])
    assert got[1]["status"] == 0 and got[1]["iterations"] == res[0]["iterations"]
