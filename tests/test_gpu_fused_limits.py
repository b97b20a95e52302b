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
