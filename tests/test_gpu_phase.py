"""Perturbation phases one iteration at a time, against the FP64 oracle's.

From the same x0 the device must try and accept the same steps (the trial
exponent ell), and its next iterate may differ by its own roundings only: g
and z to float32 (dz = 2 u (|z| + |z - x0|), which the step passes on as at
most dz + |A|^T D |A| dz), D_i, c_i and the result (2 u sum_i |c_i a_ij| +
u |x_j|), u = 2^-24.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smx():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_27086_amd as smx

    smx.lib()
    return smx


def check_iteration(smx, w, expect_launches=None):
    p = smx.problem_from_workload(w)
    if expect_launches is not None:
        assert p.describe()["phase_launches"] == expect_launches
    p.run(1)
    x = p.get_x().cpu().numpy().astype(np.float64)
    st, _ = p.get_state()
    p.close()
    u = 2.0 ** -24
    rows = np.repeat(np.arange(w.m), np.diff(w.row_ptr))
    for s in range(w.B):
        P = oracle.from_workload(w, s)
        x0 = w.x0[:, s].astype(np.float64)
        z, so = P.perturb(x0)
        assert st[s]["ell"] == so.ell, (s, st[s]["ell"], so.ell)
        xo, _ = P.step(z)
        r, q = P.matvec(z), P.row_sqnorms()
        D = np.where(q > 0, P.w / np.where(q > 0, q, 1.0), 0.0)
        c = D * (np.clip(r, P.lower, P.upper) - r)
        dz = 2 * u * (np.abs(z) + np.abs(z - x0))
        dr, terms = np.zeros(w.m), np.zeros(w.n)
        np.add.at(dr, rows, np.abs(P.val) * dz[w.col_idx])
        np.add.at(terms, w.col_idx, np.abs(P.val) * (2 * u * np.abs(c[rows]) + D[rows] * dr[rows]))
        bound = 1.01 * (terms + dz + u * np.abs(xo)) + 1e-13
        assert np.all(np.abs(x[:, s] - xo) <= bound), (s, float(np.max(np.abs(x[:, s] - xo) / bound)))
    return st


@pytest.mark.parametrize("obj,n,B,gamma,n_red", [
    (W.OBJ_SQNORM, 8200, 1, 1.0, 3),    # closed form, every first trial accepted
    (W.OBJ_SQNORM, 9000, 2, 5e3, 2),    # closed form, more rejections than one round of 64 holds
    (W.OBJ_L1, 8193, 1, 1e-4, 4),       # no entry changes sign: closed form
    (W.OBJ_L1, 10007, 1, 30.0, 4),      # signs change: trials summed
    (W.OBJ_L1, 8500, 4, 400.0, 2),      # rejected sums, several slices
    (W.OBJ_L1, 131072, 1, 300.0, 1),    # the longest x of this form
])
def test_phase_on_the_line(smx, obj, n, B, gamma, n_red):
    """Squared norm and L1 beyond n = 8,192: two launches, whose trial values
    come from f along the line.  x0 spreads over both signs with a tenth of
    its entries zero."""
    w = W.random_sparse(400, n, 10, seed=90 + n % 7, B=B, obj=obj, K=1)
    rng = np.random.default_rng(n)
    x0 = rng.uniform(-0.2, 1.0, (n, B)).astype(np.float32)
    x0[rng.random((n, B)) < 0.1] = 0.0
    w = w.with_params(gamma=gamma, alpha=0.9, n_red=n_red, x0=x0)
    check_iteration(smx, w, expect_launches=2)


def test_phase_on_the_line_ends_at_the_trial_cap(smx):
    """Every trial of the first step is rejected: the cap ends the phase and x
    stays, in closed form (squared norm) and by summation (L1)."""
    for obj in (W.OBJ_SQNORM, W.OBJ_L1):
        w = W.random_sparse(300, 8300, 10, seed=97, obj=obj, K=1).with_params(gamma=1e6, alpha=0.99, n_red=2,
                                                                             max_trials=21)
        st = check_iteration(smx, w, expect_launches=2)
        assert st[0]["trials"] == 21 and st[0]["accepts"] == 0 and st[0]["cap_hits"] == 1


@pytest.mark.parametrize("m,n", [(1, 2), (64, 17), (70, 63), (4097, 65), (16500, 324), (500, 1024), (500, 1025),
                                 (300, 2049), (200, 8192)])
def test_linear_phase_in_the_apply_kernel(smx, m, n):
    """Linear objective below n = 8,192: the phase in closed form from the
    partials that the fused pass leaves, and grids at both ends of the rule on
    rows (64 workgroups, then one for 64 rows)."""
    w = W.random_sparse(m, n, min(n, 6), seed=m, obj=W.OBJ_LINEAR, K=1)
    check_iteration(smx, w.with_params(gamma=3.0, alpha=0.9, n_red=2))


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("basic", [W.BASIC_EL, W.BASIC_EMR])
@pytest.mark.parametrize("m,n", [(5, 3), (300, 255), (300, 257), (900, 8193), (2500, 13000), (400, 30000)])
def test_linear_phase_with_extrapolated_steps(smx, m, n, basic, graph):
    """Linear objective with EL and EMR: the launch that moves x leaves the next
    phase's partials (and forms z where the pass took the phase).  Against the
    one-launch or two-launch phase: the same trials; z to one rounding, so x
    after one step to 4 units of float32 at the largest entry; and the second
    phase opens at c^T x of the first result, whose entries are rounded alike
    to one unit."""
    w = W.random_sparse(m, n, min(n, 8), seed=m, obj=W.OBJ_LINEAR, K=1)
    w = w.with_params(gamma=2.0, alpha=0.9, n_red=3, basic=basic)
    xs, ells, fs = [], [], []
    for fused in (True, False):
        p = smx.problem_from_workload(w, fused=fused, history_cap=4)
        p.run(1, graph=graph)
        xs.append(p.get_x().cpu().numpy().astype(np.float64)[:, 0])
        ells.append(p.get_state()[0][0]["ell"])
        p.reset(w.x0)
        p.run(2, graph=graph)
        h = p.history()
        fs.append(h["f_start"][:, 0])
        ells.append(tuple(h["trials"][:, 0]))
        p.close()
    u = 2.0 ** -24
    assert ells[:2] == ells[2:]
    assert np.max(np.abs(xs[0] - xs[1])) <= 8 * u * max(1.0, np.max(np.abs(xs[1])))
    c = np.asarray(w.linear_c, np.float64)
    for x, f in zip(xs, fs):
        assert abs(f[1] - c @ x) <= 2 * u * np.sum(np.abs(c * x)) + 1e-12


@pytest.mark.parametrize("obj", [W.OBJ_NONE, W.OBJ_SQNORM, W.OBJ_L1])
@pytest.mark.parametrize("B,m,n", [(1, 1, 1), (1, 5000, 3000), (8, 300, 4097), (32, 300, 200)])
def test_query_of_every_slice(smx, obj, B, m, n):
    """Both values of each slice in one launch, twice on the same problem.  The
    weights D_i are rounded to float32 (2^-24 relative) and t_i^2 is summed in
    float64; t_i = band - r_i is exact to float64 sums, so the proximity agrees
    to 2^-23 and the objective to float64 summation."""
    w = W.random_sparse(m, n, min(n, 8), seed=m + B, B=B, obj=obj, K=1)
    p = smx.problem_from_workload(w)
    for _ in range(2):
        prox, f = p.query()
        for s in range(B):
            P, x = oracle.from_workload(w, s), w.x0[:, s].astype(np.float64)
            assert abs(prox[s] - P.proximity(x)) <= 2.0 ** -23 * P.proximity(x) + 1e-18
            want = 0.0 if obj == W.OBJ_NONE else P.objective(x)
            assert abs(f[s] - want) <= 1e-12 * abs(want)
    p.close()


@pytest.mark.parametrize("B,gamma,alpha", [(1, 200.0, 0.93), (1, 3.0, 0.97), (2, 200.0, 0.93), (1, 1e6, 0.99)])
def test_tv_phase_with_failing_batches(smx, B, gamma, alpha):
    """Four reduction steps in six trial launches: first batches of 8 that fail
    (each costs its step a second launch, and after two the rest take every
    trial at once), batches that succeed, and a step that meets the cap."""
    w = W.random_sparse(900, 33 * 21, 6, seed=93, B=B, obj=W.OBJ_TV2D, K=1, tv_shape=(33, 21))
    check_iteration(smx, w.with_params(gamma=gamma, alpha=alpha, n_red=4), expect_launches=8)


@pytest.mark.parametrize("basic", [W.BASIC_SIMULT, W.BASIC_EL, W.BASIC_EMR])
@pytest.mark.parametrize("n", [700, 1500, 5000, 14000])
def test_linear_phase_is_the_same_wherever_a_run_starts(smx, n, basic):
    """The partials a run opens with are summed as those the launch that moves x
    leaves: a phase's f(x^k) has the same bits as the first of a run and inside
    one.  One row (one workgroup with entries, so that y has one order), weights
    1: three iterations in one run and in three."""
    w = W.random_sparse(1, n, n, seed=n, obj=W.OBJ_LINEAR, K=1, empty_frac=0.0, long_rows=1)
    w = w.with_params(gamma=2.0, alpha=0.9, n_red=3, basic=basic)
    got = []
    for runs in ((3,), (1, 1, 1), (2, 1)):
        p = smx.problem_from_workload(w, history_cap=4)
        for k in runs:
            p.run(k)
        h = p.history()
        got.append((h["f_start"][:, 0].tobytes(), h["f_end"][:, 0].tobytes(), p.get_x().cpu().numpy().tobytes()))
        p.close()
    assert got[0] == got[1] == got[2]


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("m,n", [(1, 2), (64, 17), (4097, 65), (16500, 324), (500, 1024), (500, 1025), (200, 8192)])
def test_second_linear_phase_opens_from_the_apply_kernel(smx, m, n, graph):
    """The partials that the fused pass's apply kernel leaves for the next phase
    (16 unknowns a workgroup to n = 1,024, 64 beyond): the second phase opens at
    c^T x of the first result, summed in float64 over float32 x, and tries as
    many steps as the two passes' second phase does."""
    w = W.random_sparse(m, n, min(n, 6), seed=m, obj=W.OBJ_LINEAR, K=1).with_params(gamma=3.0, alpha=0.9, n_red=2)
    trials = []
    for fused in (True, False):
        p = smx.problem_from_workload(w, fused=fused, history_cap=4)
        p.run(1, graph=graph)
        x = p.get_x().cpu().numpy().astype(np.float64)[:, 0]
        p.reset(w.x0)
        p.run(2, graph=graph)
        h = p.history()
        p.close()
        trials.append(tuple(h["trials"][:, 0]))
        cx = np.asarray(w.linear_c, np.float64) * x
        # the fused pass adds in no fixed order: its x may differ by a rounding from run to run
        slack = 2 * 2.0 ** -24 if fused else 1e-13
        assert abs(h["f_start"][1, 0] - cx.sum()) <= slack * np.sum(np.abs(cx)) + 1e-12
    assert trials[0] == trials[1]


@pytest.mark.parametrize("B,R,C", [(32, 64, 64), (2, 256, 256), (32, 80, 64), (16, 81, 90), (8, 130, 130),
                                   (4, 180, 181), (2, 257, 250)])
def test_tv_phase_of_several_slices(smx, B, R, C):
    """Both sides of 512 (16 x 16 tile, slice) pairs: a workgroup a slice, and
    whole lines in tiles of 2, 4, 8 and 16 rows; four steps with rejected trials."""
    w = W.random_sparse(300, R * C, 6, seed=B + R, B=B, obj=W.OBJ_TV2D, K=1, tv_shape=(R, C))
    check_iteration(smx, w.with_params(gamma=200.0, alpha=0.93, n_red=4), expect_launches=8)


@pytest.mark.parametrize("n,gamma,n_red,kind", [
    (16385, 30.0, 4, "spread"),   # the shortest sorted x: 17 chunks, one entry in the last
    (25600, 1e-4, 2, "spread"),   # no entry changes sign: closed form
    (32761, 300.0, 3, "ties"),    # three magnitudes: whole runs of equal keys
    (65536, 60.0, 1, "sparse"),   # most entries zero, the rest small
    (100003, 2e3, 4, "spread"),   # steps past the largest entry, rejected
    (131071, 100.0, 4, "spread"),
    (131072, 400.0, 2, "ties"),
])
def test_l1_phase_from_sorted_chunks(smx, n, gamma, n_red, kind):
    """L1 beyond n = 16,384: the direction launch sorts |x_j| in chunks, and a
    trial past a change of sign takes a search a chunk."""
    w = W.random_sparse(300, n, 10, seed=n % 91, obj=W.OBJ_L1, K=1)
    rng = np.random.default_rng(n)
    x0 = rng.uniform(-0.2, 1.0, (n, 1))
    if kind == "ties":
        x0 = np.array([0.0, 0.25, -0.5, 0.75])[rng.integers(0, 4, (n, 1))]
    elif kind == "sparse":
        x0 = np.where(rng.random((n, 1)) < 0.9, 0.0, 0.3 * x0 * rng.random((n, 1)))
    w = w.with_params(gamma=gamma, alpha=0.9, n_red=n_red, x0=x0.astype(np.float32))
    check_iteration(smx, w, expect_launches=2)


def test_sorted_phase_ends_at_the_trial_cap(smx):
    """Every trial rejected, in batches of eight and a rest of five."""
    w = W.random_sparse(300, 30000, 10, seed=97, obj=W.OBJ_L1, K=1).with_params(gamma=1e6, alpha=0.99, n_red=2,
                                                                               max_trials=21)
    st = check_iteration(smx, w, expect_launches=2)
    assert st[0]["trials"] == 21 and st[0]["accepts"] == 0 and st[0]["cap_hits"] == 1


@pytest.mark.parametrize("B,n,launches", [(2, 16384, 2), (2, 16385, 6), (8, 16385, 6), (16, 16384, 2),
                                          (32, 8193, 6)])
def test_l1_phase_of_several_slices(smx, B, n, launches):
    """Several slices sum past a change of sign up to n = 16,384 and 256
    workgroups, then take the chain."""
    w = W.random_sparse(200, n, 8, seed=B, B=B, obj=W.OBJ_L1, K=1)
    check_iteration(smx, w.with_params(gamma=40.0, alpha=0.9, n_red=2), expect_launches=launches)


def test_footprint_counts_the_sorted_chunks(smx):
    """16,385 unknowns allocate what the plan says, with the chunks' buffer."""
    w = W.random_sparse(100, 16385, 5, seed=4, obj=W.OBJ_L1, K=1)
    p = smx.problem_from_workload(w)
    got = p.describe()["device_bytes"]
    p.close()
    _, plan = smx.problem_footprint(w.m, w.n, len(w.val), "f32", obj=W.OBJ_L1)
    assert got == plan
    _, short = smx.problem_footprint(w.m, 16384, len(w.val), "f32", obj=W.OBJ_L1)
    assert plan - short >= 17 * (1024 * 4 + 32 * 12)


@pytest.mark.parametrize("obj,n", [(W.OBJ_SQNORM, 9000), (W.OBJ_L1, 9000), (W.OBJ_L1, 20000)])
def test_adaptive_step_on_the_line(smx, obj, n):
    """The adaptive step has one trial a phase, whose step no window holds: four
    iterations on the line and by the chain take the same ones.  x0 is near 0, so
    that the steps T raise f and every later phase has its trial.  The passes
    of both are the bitwise ones and f agrees to float64 summation, so an
    iteration moves an entry by a float32 rounding of z and of x, which T passes
    on as they are: 8 u of the largest entry after four, u = 2^-24, and twice
    that of f relative to the sum of |x_j| or x_j^2."""
    w = W.random_sparse(500, n, 12, seed=n % 83, obj=obj, K=1)
    rng = np.random.default_rng(n)
    w = w.with_params(x0=(0.02 * rng.uniform(-1.0, 1.0, (n, 1))).astype(np.float32))
    got = []
    for form in (smx.PHASE_AUTO, smx.PHASE_BATCHES):
        p = smx.problem_from_workload(w, fused=False, history_cap=8, step_rule=1)
        p.set_phase_form(form)
        p.run(4)
        h = p.history()
        got.append((tuple(h["trials"][:, 0]), tuple(h["accepts"][:, 0]), h["f_start"][:, 0].copy(),
                    p.get_x().cpu().numpy().astype(np.float64)))
        p.close()
    assert got[0][:2] == got[1][:2] and sum(got[0][0]) >= 2
    u = 2.0 ** -24
    assert np.all(np.abs(got[0][2] - got[1][2]) <= 32 * u * np.abs(got[1][2]))
    assert np.max(np.abs(got[0][3] - got[1][3])) <= 8 * u * max(1.0, np.max(np.abs(got[1][3])))
