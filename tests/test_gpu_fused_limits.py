"""The fused pass where its LDS is full: 160 KB hold 12 bytes an unknown (z and
a float64 y) up to n = 13,568, 8 (z and a float32 y, or a float64 y alone) up to
20,352, beside the kernel's own arrays.  Up to the last of them the pass is
taken, in each shape that fits.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

EDGES = [13556, 13557, 13568, 13569, 20332, 20333, 20352, 20353]


@pytest.fixture(scope="module")
def smx():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_27086_amd as smx

    smx.lib()
    return smx


def close_to(got, want):
    """One step from the same x0: z and x are rounded to float32 on each path
    (4 u), and a float32 y adds at most eight terms a column and workgroup, whose
    sum is under 1/2 (uniform weights 1/m): 4 u more, u = 2^-24."""
    return np.max(np.abs(got - want)) <= 8 * 2.0 ** -24 * max(1.0, float(np.max(np.abs(want))))


@pytest.mark.parametrize("n", EDGES)
def test_every_shape_that_fits_runs(smx, n):
    """Linear objective, phase inside the pass where z is in LDS, against the
    two passes: the same trials, x to its roundings."""
    w = W.random_sparse(300, n, 8, seed=n % 97, obj=W.OBJ_LINEAR, K=1).with_params(gamma=2.0, alpha=0.9, n_red=2)
    ref = smx.problem_from_workload(w, fused=False)
    ref.run(1)
    want, ell = ref.get_x().cpu().numpy().astype(np.float64), ref.get_state()[0][0]["ell"]
    ref.close()
    p = smx.problem_from_workload(w)
    info = p.describe()["f32"]["fused"]
    assert info is not None and info["in_use"]
    assert info["zl"] == (1 if n <= 13568 else 0)
    shapes = [None, (8, 4, 0, 0)]
    if n <= 20352:
        shapes += [(8, 4, 0, 1), (16, 8, 2, 1)]
    else:
        with pytest.raises(smx.SmxError):
            p.set_fused_shape(8, 4, 0, 1)
    for shape in shapes:
        if shape is not None:
            p.set_fused_shape(*shape)
        p.reset(w.x0)
        p.run(1)
        assert p.get_state()[0][0]["ell"] == ell, shape
        assert close_to(p.get_x().cpu().numpy().astype(np.float64), want), shape
    p.close()


@pytest.mark.parametrize("n", EDGES)
def test_dose_volume_rows_keep_the_pass(smx, n):
    """Dose-volume rows need z in LDS: the fused pass up to 20,352 unknowns."""
    w = W.random_sparse(300, n, 8, seed=n % 89, obj=W.OBJ_NONE, K=1)
    w = w.with_params(dvc=[dict(row_begin=180, row_end=300, sense=W.DVC_MAX, fraction=0.3, dose=0.1)])
    xs = []
    for fused in (True, False):
        p = smx.problem_from_workload(w, fused=fused)
        info = p.describe()["f32"]["fused"]
        if n <= 20352:
            assert info is not None and info["in_use"] == fused and info["zl"] == 1
        else:
            assert info is None
        p.run(1, perturb=False)
        xs.append(p.get_x().cpu().numpy().astype(np.float64))
        p.close()
    assert close_to(xs[0], xs[1])


@pytest.mark.parametrize("n,shape", [(900, (8, 4, 0, 1)), (900, (8, 4, 0, 0)), (900, (16, 4, 4, 0)),
                                     (14000, (8, 4, 0, 1)), (14000, (16, 8, 2, 1)), (21000, (8, 4, 0, 0)),
                                     (21000, (16, 8, 0, 0)), (21000, (16, 4, 4, 0))])
def test_infinite_row_reaches_its_columns_alone(smx, n, shape):
    """A row whose value is -inf has c = +inf: its columns go to the box's upper
    bound, the one at its end too, which the padding behind the row (value 0)
    names again, and a stored zero adds nothing.  The other columns are those
    of the same x0 without the infinity."""
    rng = np.random.default_rng(n)
    m, own = 70, np.array([5, 9, 11, 20])
    cols = [np.sort(rng.choice(np.setdiff1d(np.arange(n), own), size=1 + i % 11, replace=False)) for i in range(m)]
    cols[7] = np.array([5, 20, 9, 11])
    ptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    col = np.concatenate(cols).astype(np.int32)
    val = rng.uniform(0.5, 1.5, len(col)).astype(np.float32)
    val[col == 20] = 0.0
    x0 = rng.uniform(0.1, 1.0, (n, 1)).astype(np.float32)
    w = W.Workload(name="inf", m=m, n=n, row_ptr=ptr, col_idx=col, val=val, lower=np.full((m, 1), -0.1, np.float32),
                   upper=np.full((m, 1), 0.1, np.float32), x0=x0, box_lo=np.full(n, -1e30, np.float32),
                   box_hi=np.full(n, 1e30, np.float32), lam=1.0, K=1)
    ref = smx.problem_from_workload(w, fused=False)
    ref.run(1, perturb=False)
    want = ref.get_x().cpu().numpy().astype(np.float64)[:, 0]
    ref.close()
    p = smx.problem_from_workload(w)
    p.set_fused_shape(*shape)
    x0[5] = -np.inf
    p.set_x(x0)
    p.run(1, perturb=False)
    got = p.get_x().cpu().numpy().astype(np.float64)[:, 0]
    p.close()
    rest = np.setdiff1d(np.arange(n), [5, 9, 11])
    assert got[9] == got[11] == np.float32(1e30)
    assert close_to(got[rest], want[rest])


def test_pinned_shape_takes_the_larger_grid(smx):
    """Up to 2,048 columns the tuner tries a shape with z in LDS at two grids;
    a shape that is asked for by name gets the one of the default shape, as many
    workgroups as the rows use, again and again."""
    w = W.random_sparse(20000, 300, 4, seed=5, obj=W.OBJ_NONE, K=1)
    p = smx.problem_from_workload(w)
    grid = p.describe()["f32"]["fused"]["grid"]
    assert grid == 313  # ceil(20000 / 64), over one workgroup a CU
    for shape in ((8, 8, 0, 1), (8, 4, 0, 0), (16, 4, 4, 1), (32, 8, 2, 1), (16, 8, 2, 1)):
        p.set_fused_shape(*shape)
        assert p.describe()["f32"]["fused"]["grid"] == grid, shape
    p.close()


@pytest.mark.parametrize("n,dvc,kind,vectors,columns", [
    (900, False, "f64", 64, 16), (1025, False, "f64", 64, 64), (900, True, "f32", 65, 16),
    (13569, True, "f32", 65, 64), (21000, False, "f32", 64, 64),
])
def test_describe_names_the_partial_vectors(smx, n, dvc, kind, vectors, columns):
    """What the launch after the fused pass sums: float64 vectors from a float64
    y, float32 ones from a float32 y and wherever dose-volume rows add theirs
    (here one more), 16 or 64 columns a workgroup; the benchmark's byte count
    and kernel name go by it."""
    import bench

    w = W.random_sparse(300, n, 8, seed=n % 89, obj=W.OBJ_NONE, K=1)
    if dvc:
        w = w.with_params(dvc=[dict(row_begin=180, row_end=300, sense=W.DVC_MAX, fraction=0.3, dose=0.1)])
    p = smx.problem_from_workload(w)
    shapes = p.describe()["f32"]
    p.close()
    assert shapes["fused"]["partials"] == dict(type=kind, vectors=vectors, columns=columns)
    size, name = (8, "double") if kind == "f64" else (4, "float")
    assert bench.alg_bytes(w.m, n, w.nnz, shapes)[1] == size * n * vectors + 16 * n
    assert bench.kernel_name(2, shapes["pass2"], 1, shapes) == f"smx::k_fused_apply<{name}, {columns}>"
