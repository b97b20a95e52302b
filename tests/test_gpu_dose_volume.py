"""Selection of dose-volume constraints with many equal values: equal values
rank by row, across the workgroups of a constraint."""
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


def _ties(B, fractions, seed):
    """9,400 single-entry rows of value 1 on 11 columns (so a row's value is an
    entry of x) with random weights, all in two constraints of 7,000 and 2,100
    rows beside 300 plain bands.  The columns hold four distinct values, some
    equal in float32 only after rounding, one column for all rows of slice 1."""
    rng = np.random.default_rng(seed)
    n, n0, n1, n2 = 11, 300, 7000, 2100
    m = n0 + n1 + n2
    col = rng.integers(0, n, m).astype(np.int32)
    x0 = np.empty((n, B), np.float32)
    x0[:, 0] = np.array([0.25, 0.5, 0.5, 0.75, 1.0])[rng.integers(0, 5, n)]
    if B > 1:
        x0[:, 1] = 0.5  # every row ties
    w = W.Workload(
        name="ties", m=m, n=n, row_ptr=np.arange(m + 1, dtype=np.int32), col_idx=col, val=np.ones(m, np.float32),
        lower=np.full((m, B), 0.6, np.float32), upper=np.full((m, B), 0.7, np.float32), x0=x0,
        box_lo=np.full(n, -np.inf, np.float32), box_hi=np.full(n, np.inf, np.float32), lam=1.0, K=1,
        weights=rng.uniform(0.5, 2.0, m))
    return w.with_params(dvc=[
        dict(row_begin=n0, row_end=n0 + n1, sense=W.DVC_MAX, fraction=fractions[0], dose=0.2),
        dict(row_begin=n0 + n1, row_end=m, sense=W.DVC_MIN, fraction=fractions[1], dose=1.5)])


@pytest.mark.parametrize("B,fused", [(1, True), (1, False), (2, False)])
@pytest.mark.parametrize("fractions", [(0.37, 0.41), (0.0, 1.0), (1.0, 0.0), (0.9999, 0.0001)])
def test_ties_rank_by_row(smx, B, fused, fractions):
    """One step and the proximity against the oracle: 2 u sum_i |c_i a_ij| + u
    |x_j| (u = 2^-24: D_i, c_i and the result are float32) separate two rows'
    weights many times over; k of each constraint falls among equal values,
    takes none, all, all but one and one of the rows."""
    w = _ties(B, fractions, seed=101)
    p = smx.problem_from_workload(w, fused=fused)
    prox, _ = p.query()
    p.run(1, perturb=False)
    x = p.get_x().cpu().numpy().astype(np.float64)
    p.run(1, perturb=False)  # the scratch is left as it was found
    y = p.get_x().cpu().numpy().astype(np.float64)
    p.set_x(w.x0)
    p.run(1, perturb=False)
    again = p.get_x().cpu().numpy().astype(np.float64)
    p.close()
    u = 2.0 ** -24
    for s in range(B):
        P = oracle.from_workload(w, s)
        x0 = w.x0[:, s].astype(np.float64)
        xo, po = P.step(x0)
        assert abs(prox[s] - po) <= 4 * u * po
        lo, up = P.bands_at(x0)
        r = P.matvec(x0)
        c = P.w * (np.clip(r, lo, up) - r)  # ||a_i|| = 1
        terms = np.zeros(w.n)
        np.add.at(terms, w.col_idx, np.abs(c))
        for got in (x[:, s], again[:, s]):
            assert np.all(np.abs(got - xo) <= 1.01 * (2 * u * terms + u * np.abs(xo)) + 1e-13)
        assert np.all(np.isfinite(y[:, s]))


@pytest.mark.parametrize("fused", [True, False])
def test_more_chunks_of_rows_than_workgroups(smx, fused):
    """1.1 million rows in two constraints: 538 chunks of 2,048 rows, more than
    the fused pass's workgroups (512 here), whose partials the band kernel's add
    to, so that some take two chunks, of both constraints.  Bounds as above."""
    rng = np.random.default_rng(7)
    n, n0, n1, n2 = 13, 500, 700_001, 400_000
    m = n0 + n1 + n2
    w = W.Workload(
        name="chunks", m=m, n=n, row_ptr=np.arange(m + 1, dtype=np.int32), col_idx=rng.integers(0, n, m).astype(np.int32),
        val=rng.uniform(0.5, 1.5, m).astype(np.float32), lower=np.full((m, 1), 0.6, np.float32),
        upper=np.full((m, 1), 0.7, np.float32), x0=rng.uniform(0.2, 1.0, (n, 1)).astype(np.float32),
        box_lo=np.full(n, -np.inf, np.float32), box_hi=np.full(n, np.inf, np.float32), lam=1.0, K=1,
        weights=rng.uniform(0.5, 2.0, m))
    w = w.with_params(dvc=[dict(row_begin=n0, row_end=n0 + n1, sense=W.DVC_MAX, fraction=0.37, dose=0.4),
                           dict(row_begin=n0 + n1, row_end=m, sense=W.DVC_MIN, fraction=0.41, dose=1.1)])
    p = smx.problem_from_workload(w, fused=fused)
    if fused:
        assert p.describe()["f32"]["fused"]["grid"] < 538
    prox, _ = p.query()
    got = []
    for _ in range(2):
        p.set_x(w.x0)
        p.run(1, perturb=False)
        got.append(p.get_x().cpu().numpy().astype(np.float64)[:, 0])
    p.close()
    u = 2.0 ** -24
    P, x0 = oracle.from_workload(w, 0), w.x0[:, 0].astype(np.float64)
    xo, po = P.step(x0)
    assert abs(prox[0] - po) <= 4 * u * po
    lo, up = P.bands_at(x0)
    r = P.matvec(x0)
    c = P.w / P.row_sqnorms() * (np.clip(r, lo, up) - r)
    terms = np.zeros(n)
    np.add.at(terms, w.col_idx, np.abs(c * P.val))
    for x in got:
        assert np.all(np.abs(x - xo) <= 1.01 * (2 * u * terms + u * np.abs(xo)) + 1e-13)
