"""Short-row solves run as one launch of resident workgroups: sizes around the
edges of its tiles (512 rows), of its exchange (up to 32 workgroups read all
partial sums, above one workgroup sums a column) and of its split of a tile
over 8, 4 and 2 waves, a row block with more entries than its staging
buffer, and restarts so short that a solve takes several launches.

The matrix has a diagonal of 4 and off-diagonals whose absolute sum is at most
2 a row, so ||A^-1|| <= 1/2 and ||A|| <= 6 in the infinity norm; two iterates with relative residuals
of at most 1e-10 differ by at most 2 kappa 1e-10 = 6e-10 there, and by at most
that times sqrt(n) / 1 in the 2-norm relative to ||x|| for entries of like
size; 1e-8 is asked for."""
import ctypes as C
import time

import numpy as np
import pytest

import oracle
import paper_2409_15468_amd as cb
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def near_diagonal(n, seed, wide_row=None):
    """Rows of 4 on the diagonal with up to four neighbours at distances 1 and
    37; row wide_row (if given) has 600 entries of 1/600."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    offs = np.array([-37, -1, 0, 1, 37])
    cols = i[:, None] + offs
    vals = rng.uniform(-0.5, 0.5, cols.shape)
    vals[:, 2] = 4.0
    keep = (cols >= 0) & (cols < n)
    rows = np.broadcast_to(i[:, None], cols.shape)[keep]
    c, v = cols[keep], vals[keep]
    if wide_row is not None:
        off = rows != wide_row
        wide = np.unique(np.append(rng.choice(n, 600, replace=False), wide_row))
        wv = np.full(wide.size, 1.0 / 600)
        wv[wide == wide_row] = 4.0
        at = np.searchsorted(rows, wide_row)
        rows = np.concatenate([rows[:at], np.full(wide.size, wide_row), rows[at:][off[at:]]])
        c = np.concatenate([c[:at], wide, c[at:][off[at:]]])
        v = np.concatenate([v[:at], wv, v[at:][off[at:]]])
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return synth.CSR(n, rp, c.astype(np.int32), np.ascontiguousarray(v))


def check(A, m, fmt, seed, history_cap=1000):
    b = A.scipy() @ np.random.default_rng(seed).uniform(-1, 1, A.n)
    xd = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    print(f"n={A.n} m={m} {fmt}", flush=True)
    res, hist = cb.cbgmres_solve(cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val), torch.from_numpy(b).cuda(), xd, m,
                                 1e-10, fmt, history_cap=history_cap)
    x = xd.cpu().numpy()
    ref = oracle.gmres(A, b, m, 1e-10, fmt, hist_cap=history_cap)
    assert res["status"] == 0 and res["converged"]
    assert np.linalg.norm(b - A.scipy() @ x) <= 1e-10 * (1 + 1e-6) * np.linalg.norm(b)
    assert np.linalg.norm(x - ref.x) <= 1e-8 * np.linalg.norm(ref.x)
    assert abs(res["iterations"] - ref.iterations) <= max(1, int(0.02 * ref.iterations))
    assert hist.size == min(history_cap, res["iterations"])
    k = min(5, hist.size)
    np.testing.assert_allclose(hist[:k], ref.history[:k], rtol=1e-3)  # 64 steps of a 16-bit code at most
    return res, x


@pytest.mark.parametrize("n,fmt", [(1, "float64"), (31, "frsz2_32"), (511, "frsz2_16"), (512, "frsz2_21"), (513, "frsz2_32"),
                                   (4097, "float32"), (16384, "frsz2_32"), (16385, "frsz2_32"), (16385, "frsz2_21"),
                                   (131072, "frsz2_32"), (131073, "frsz2_16"), (131073, "float64"), (262145, "frsz2_32"),
                                   (262145, "float64"), (524289, "frsz2_32"), (1048576, "float32"), (1048577, "frsz2_32")])
def test_edges(n, fmt):
    check(near_diagonal(n, n), 30, fmt, n + 1)


@pytest.mark.parametrize("n", [700, 20000])
def test_long_row(n):
    check(near_diagonal(n, n, wide_row=n // 3), 30, "frsz2_32", n)


@pytest.mark.parametrize("n,width,count", [(3000, 2999, 1), (700, 257, 1), (20000, 9000, 3), (400, 399, 400)])
def test_rows_longer_than_the_staging_buffer(n, width, count):
    """One row with most of its block's entries (staged in pieces of 256), in a
    block of other long rows (a lane per row), and a dense matrix, alone and as a
    batch, against the oracle's iterations and x."""
    A = near_diagonal(n, n)
    rng = np.random.default_rng(n)
    M = A.scipy().tolil()
    for r in rng.choice(n, count, replace=False):
        c = rng.choice(n, width, replace=False)
        M[r, c] = rng.uniform(-1, 1, width) / width
        M[r, r] = 4.0
    M = M.tocsr()
    M.sort_indices()
    A = synth.CSR(n, M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data)
    b = M @ rng.uniform(-1, 1, n)
    ref = oracle.gmres(A, b, 30, 1e-10, "frsz2_32")
    Ad, bd = cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val), torch.from_numpy(b).cuda()
    for batch in (False, True):
        print(f"long rows n={n} width={width} count={count} batch={batch}", flush=True)
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        if batch:
            res = cb.cbgmres_solve_batch([(Ad, bd, x, 30, 1e-10, "frsz2_32")])[0]
        else:
            res, _ = cb.cbgmres_solve(Ad, bd, x, 30, 1e-10, "frsz2_32")
        assert res["converged"] and abs(res["iterations"] - ref.iterations) <= 1
        assert np.linalg.norm(x.cpu().numpy() - ref.x) <= 1e-8 * np.linalg.norm(ref.x)
        assert np.linalg.norm(b - M @ x.cpu().numpy()) <= 1e-10 * (1 + 1e-6) * np.linalg.norm(b)


@pytest.mark.parametrize("m", [1, 2, 3, 104, 105])
def test_restart_lengths(m):
    """A launch ends when the next cycle's history might not fit in m (m + 1)
    entries: with m = 1, 2, 3 these solves take several.  104 is the longest
    restart the team takes."""
    res, x = check(near_diagonal(3000, m), m, "frsz2_32", m)
    again, y = check(near_diagonal(3000, m), m, "frsz2_32", m, history_cap=0)
    assert again["iterations"] == res["iterations"] and np.array_equal(x, y)


def test_batch_over_several_launches():
    """Five systems of the batch's largest size take more workgroups than the
    GPU has CUs, so the batch runs as several launches; small ones (one and two
    tiles, the change from 8 to 4 waves a tile) fill the gaps.  Every result is
    that of the system alone, bit for bit, and meets its tolerance."""
    sizes = [65536, 512, 65000, 513, 1, 65536, 1025, 64513, 65536, 3000]
    formats = ["frsz2_32", "float64", "frsz2_21", "float32", "frsz2_16", "float16"]
    systems, rhs = [], []
    for i, n in enumerate(sizes):
        A = near_diagonal(n, i)
        b = A.scipy() @ np.random.default_rng(100 + i).uniform(-1, 1, n)
        rhs.append((A, b))
        systems.append((cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val), torch.from_numpy(b).cuda(),
                        torch.zeros(n, dtype=torch.float64, device="cuda"), 20, 1e-10, formats[i % 6]))
    print("batch", flush=True)
    res = cb.cbgmres_solve_batch(systems)
    for i, (s, (A, b)) in enumerate(zip(systems, rhs)):
        x = s[2].cpu().numpy()
        assert res[i]["converged"]
        assert np.linalg.norm(b - A.scipy() @ x) <= 1e-10 * (1 + 1e-6) * np.linalg.norm(b)
        alone = s[:2] + (torch.zeros_like(s[2]),) + s[3:]
        r = cb.cbgmres_solve_batch([alone])[0]
        assert r["iterations"] == res[i]["iterations"]
        assert np.array_equal(alone[2].cpu().numpy(), x), sizes[i]


def test_batch_keeps_x_of_a_cycle_that_overflows():
    """Row 5 of I + L has an entry of 1e200, which step 5 from b = e_0 meets: the
    norm overflows, and x is still what the cycle began with, with and without
    teams."""
    n = 600
    i = np.arange(n)
    col = np.concatenate([[0], np.stack([i[:-1], i[1:]], 1).ravel()]).astype(np.int32)
    val = np.ones(col.size)
    val[1 + 2 * 4] = 1e200  # (5, 4)
    rp = np.concatenate([[0], 2 * i + 1]).astype(np.int32)
    Ad = cb.DeviceCSR.from_host(rp, col, val)
    b = torch.zeros(n, dtype=torch.float64, device="cuda")
    b[0] = 1.0
    for wait in (-1, 0):
        cb.lib().cb_internal_team_wait(wait, 0)
        try:
            x = torch.zeros(n, dtype=torch.float64, device="cuda")
            r = cb.cbgmres_solve_batch([(Ad, b, x, 30, 1e-10, "float64")])[0]
        finally:
            cb.lib().cb_internal_team_wait(-1, 0)
        assert r["status"] == cb.CB_ERR_NONFINITE and r["iterations"] == 4 and r["restarts"] == 1
        assert r["rel_residual"] == 1.0 and not x.any()


def test_batch_does_not_wait_for_its_slow_systems_in_turn():
    """1280 one-workgroup systems, five times what the GPU holds, of which every
    256th runs 2000 steps (a tolerance it cannot meet): the slow ones run side by
    side.  One after the other they would take five times what they take alone;
    less than half of that is asked for."""
    A = synth.convection_diffusion(20, 2, (20.0, 0.0))
    b = torch.from_numpy(synth.rhs_from_solution(A, np.random.default_rng(1).uniform(-1, 1, A.n))).cuda()
    Ad = cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val)

    def run(tols):
        x = torch.zeros((len(tols), A.n), dtype=torch.float64, device="cuda")
        size = cb.cbgmres_batch_workspace_bytes(A.n, 30, "frsz2_32")
        ws = [torch.empty(size, dtype=torch.uint8, device="cuda") for _ in tols]
        best = 1e9
        for _ in range(3):
            x.zero_()
            torch.cuda.synchronize()
            t = time.perf_counter()
            res = cb.cbgmres_solve_batch([(Ad, b, xi, 30, tol, "frsz2_32") for xi, tol in zip(x, tols)], workspaces=ws,
                                         max_iters=2000)
            best = min(best, time.perf_counter() - t)
        return best, res, x

    slow, _, _ = run([1e-30] * 5)
    mixed, res, x = run([1e-30 if i % 256 == 7 else 1e-6 for i in range(1280)])
    print(f"slow ones alone {slow * 1e3:.1f} ms, mixed {mixed * 1e3:.1f} ms", flush=True)
    assert mixed < 2.5 * slow
    assert all(r["iterations"] == 2000 if i % 256 == 7 else r["converged"] for i, r in enumerate(res))
    assert torch.equal(x[0].expand(1280, -1)[:7], x[:7]) and torch.equal(x[0], x[1279])


@pytest.mark.parametrize("fmt", ["float64", "frsz2_32"])
@pytest.mark.parametrize("eta", [None, 0.2])
def test_basis_bytes_are_those_of_the_other_paths(fmt, eta):
    """The count of passes over the columns does not depend on how a solve is
    launched: a team, or one launch per operation (m = 3 with a history: several
    launches of a team); with eta = 0.2 few steps ask for the second pass, so a
    cycle of fused updates is followed by separate ones."""
    kw = {} if eta is None else {"eta": eta}
    A = synth.convection_diffusion(40, 2, (20.0, 0.0))
    b = torch.from_numpy(synth.rhs_from_solution(A, np.random.default_rng(2).uniform(-1, 1, A.n))).cuda()
    Ad = cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val)

    def run(m, iters, wait, batch=False):
        cb.lib().cb_internal_team_wait(wait, 0)
        try:
            x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
            if batch:
                return cb.cbgmres_solve_batch([(Ad, b, x, m, 1e-14, fmt)], max_iters=iters, **kw)[0]
            return cb.cbgmres_solve(Ad, b, x, m, 1e-14, fmt, max_iters=iters, history_cap=100, **kw)[0]
        finally:
            cb.lib().cb_internal_team_wait(-1, 0)

    for m, iters in ((3, 40), (25, 70)):
        for batch in (False, True):
            team, other = run(m, iters, -1, batch), run(m, iters, 0, batch)
            print(fmt, eta, m, batch, team["reorths"], team["basis_bytes"], flush=True)
            assert team["iterations"] == other["iterations"] == iters
            assert team["reorths"] == other["reorths"] and team["basis_bytes"] == other["basis_bytes"]


@pytest.mark.parametrize("fuse", [1, 2])
def test_fuse_updates_asks_for_the_launches(fuse):
    """fuse_updates 1 and 2: bit for bit the solve without teams, and by their
    own count of passes (separate: 2 + 2 per second pass, fused: 3 + 1)."""
    A = synth.convection_diffusion(40, 2, (20.0, 0.0))
    b = torch.from_numpy(synth.rhs_from_solution(A, np.random.default_rng(2).uniform(-1, 1, A.n))).cuda()
    Ad = cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val)
    got = []
    for wait in (-1, 0):
        cb.lib().cb_internal_team_wait(wait, 0)
        try:
            x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
            got.append((cb.cbgmres_solve(Ad, b, x, 30, 1e-14, "float64", max_iters=30, fuse_updates=fuse, eta=0.2)[0], x))
        finally:
            cb.lib().cb_internal_team_wait(-1, 0)
    (r, x), (r0, x0) = got
    assert torch.equal(x, x0) and r["basis_bytes"] == r0["basis_bytes"]
    assert r["reorths"] < 30
    columns = sum(range(1, 31))
    least = (3 if fuse == 2 else 2) * columns + 30
    passes = r["basis_bytes"] / (cb.cb_basis_column_bytes("float64", A.n))
    assert passes == least if r["reorths"] == 0 else least < passes < 4 * columns + 30


def test_every_ordinary_stream_has_teams():
    """The same bits on the default stream and on another one, and other bits
    than where no team forms."""
    A = near_diagonal(20000, 3)
    b = torch.from_numpy(A.scipy() @ np.random.default_rng(7).uniform(-1, 1, A.n)).cuda()
    Ad = cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val)

    def run():
        x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        assert cb.cbgmres_solve(Ad, b, x, 30, 1e-10, "float32")[0]["converged"]
        torch.cuda.synchronize()
        return x

    first = run()
    with torch.cuda.stream(torch.cuda.Stream()):
        assert torch.equal(run(), first)
    cb.lib().cb_internal_team_wait(0, 0)
    try:
        assert not torch.equal(run(), first)
    finally:
        cb.lib().cb_internal_team_wait(-1, 0)


def test_stream_that_may_use_half_the_cus():
    """On a stream with a CU mask no team is tried: the solve and the batch take
    their other paths at once (within half the time that a team is waited for)."""
    hip = cb.lib()  # (its HIP runtime)
    torch.zeros(1, device="cuda")
    words = -(-torch.cuda.get_device_properties(0).multi_processor_count // 32)
    mask = (C.c_uint32 * words)(*[0x55555555] * words)
    h = C.c_void_p()
    if hip.hipExtStreamCreateWithCUMask(C.byref(h), words, mask) != 0:
        hip.hipGetLastError()  # or the next call reports it
        pytest.skip("the driver here makes no streams with a CU mask")
    A = near_diagonal(131072, 4)
    b = A.scipy() @ np.random.default_rng(5).uniform(-1, 1, A.n)
    small = near_diagonal(3000, 4)
    bs = small.scipy() @ np.random.default_rng(6).uniform(-1, 1, small.n)
    stream = torch.cuda.ExternalStream(h.value)
    try:
        with torch.cuda.stream(stream):
            Ad, As = (cb.DeviceCSR.from_host(M.row_ptr, M.col, M.val) for M in (A, small))
            bd, bsd = torch.from_numpy(b).cuda(), torch.from_numpy(bs).cuda()
            for _ in range(2):
                x, xs = (torch.zeros(M.n, dtype=torch.float64, device="cuda") for M in (A, small))
                stream.synchronize()
                t = time.perf_counter()
                res, _ = cb.cbgmres_solve(Ad, bd, x, 30, 1e-10, "frsz2_32")
                t1 = time.perf_counter()
                rb = cb.cbgmres_solve_batch([(As, bsd, xs, 30, 1e-10, "frsz2_32")])[0]
                t2 = time.perf_counter()
                print(f"solve {t1 - t:.4f} s, batch {t2 - t1:.4f} s", flush=True)
            assert t1 - t < 0.05 and t2 - t1 < 0.05
            for M, rhs, sol, r in ((A, b, x, res), (small, bs, xs, rb)):
                assert r["converged"]
                assert np.linalg.norm(rhs - M.scipy() @ sol.cpu().numpy()) <= 1e-10 * (1 + 1e-6) * np.linalg.norm(rhs)
            stream.synchronize()
    finally:
        torch.cuda.synchronize()
        assert hip.hipStreamDestroy(h) == 0


def test_a_thousand_small_requests_in_flight():
    """1000 requests that run 20000 steps each (a tolerance they cannot meet):
    the device-resident loop takes them all at once, and ends them all."""
    A = synth.convection_diffusion(4, 2, (20.0, 0.0))
    b = synth.rhs_from_solution(A, np.random.default_rng(1).uniform(-1, 1, A.n))
    srv = cb.Server(4 << 30, 0, lanes=1)
    tickets = [srv.submit(A.row_ptr, A.col, A.val, b, 2, 1e-30, "float64") for _ in range(1000)]
    running, t0, got = 0, time.time(), {}
    while len(got) < len(tickets) and time.time() - t0 < 60:
        running = max(running, srv.stats()[2])
        for t in tickets:
            if t not in got and (r := srv.poll(t, A.n)) is not None:
                got[t] = r
        time.sleep(0.002)
    srv.close()
    print(f"{running} at once, {time.time() - t0:.2f} s", flush=True)
    assert len(got) == 1000 and running > 900
    assert {(r[1]["status"], r[1]["iterations"]) for r in got.values()} == {(cb.CB_ERR_NOT_CONVERGED, 20000)}


def test_a_team_that_is_lost():
    """A row of some 10^5 entries keeps one workgroup at its product for
    milliseconds.  With a limit of 0 on the exchanges the others give up waiting
    (every kernel ends by itself): the solve, the batch and a served request go
    to their other paths with x as it was, and give those paths' bits."""
    rng = np.random.default_rng(3)
    for kind, n in (("solve", 100000), ("batch", 60000), ("served", 16000)):
        A = near_diagonal(n, n)
        M = A.scipy().tolil()
        c = rng.choice(n, n - n // 8, replace=False) if kind != "served" else np.arange(n)
        M[n // 3, c] = rng.uniform(-1, 1, c.size) / c.size
        M[n // 3, n // 3] = 4.0
        M = M.tocsr()
        M.sort_indices()
        A = synth.CSR(n, M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data)
        b, x0 = M @ rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
        Ad, bd = cb.DeviceCSR.from_host(A.row_ptr, A.col, A.val), torch.from_numpy(b).cuda()
        got = []
        for wait, poll in ((-1, 0), (0, -1)):
            print(f"{kind} wait {wait} poll {poll}", flush=True)
            cb.lib().cb_internal_team_wait(wait, 0)
            cb.lib().cb_internal_team_poll(poll)
            try:
                if kind == "served":
                    srv = cb.Server(4 << 30, 0, lanes=1)
                    t = srv.submit(A.row_ptr, A.col, A.val, b, 20, 1e-10, "frsz2_32", x0=x0)
                    t0, r = time.time(), None
                    while r is None and time.time() - t0 < 20:
                        time.sleep(0.001)
                        r = srv.poll(t, n)
                    srv.close()
                    x, res = r[0], r[1]
                else:
                    xd = torch.from_numpy(x0.copy()).cuda()
                    if kind == "solve":
                        res, _ = cb.cbgmres_solve(Ad, bd, xd, 20, 1e-10, "frsz2_32")
                    else:
                        res = cb.cbgmres_solve_batch([(Ad, bd, xd, 20, 1e-10, "frsz2_32")])[0]
                    x = xd.cpu().numpy()
            finally:
                cb.lib().cb_internal_team_wait(-1, 0)
                cb.lib().cb_internal_team_poll(-1)
            assert res["status"] == 0 and res["converged"]
            assert np.linalg.norm(b - M @ x) <= 1e-10 * (1 + 1e-6) * np.linalg.norm(b)
            got.append((x, res["iterations"], res["restarts"]))
        if kind != "served":  # (16000 entries may not take long enough to lose a team)
            assert np.array_equal(got[0][0], got[1][0]) and got[0][1:] == got[1][1:]


def test_served_small_then_large():
    """A small request starts the serving launch (128 workgroups); the larger
    ones after it need 138 and 256 of the GPU's CUs, so they run only if
    that launch gives its CUs back, and the last small one only if they do."""
    srv = cb.Server(8 << 30, 0, lanes=2)
    for i, n in enumerate([900, 70000, 131072, 901]):
        A = near_diagonal(n, i)
        b = A.scipy() @ np.random.default_rng(200 + i).uniform(-1, 1, n)
        print(f"serve n={n}", flush=True)
        t = srv.submit(A.row_ptr, A.col, A.val, b, 20, 1e-10, "frsz2_32")
        t0, got = time.time(), None
        while got is None and time.time() - t0 < 20:
            time.sleep(0.001)
            got = srv.poll(t, n)
        assert got is not None, "not served"
        x = got[0]
        assert np.linalg.norm(b - A.scipy() @ x) <= 1e-10 * (1 + 1e-6) * np.linalg.norm(b)
    srv.close()
