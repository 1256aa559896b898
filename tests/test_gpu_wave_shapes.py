"""The wave-per-cell integrator at the edges of its built shapes: row counts
(16, 24, 36, 48, 64 rows of N = K + 1 unknowns), reactions per lane (up to
64, 128 and 256 reactions in registers, more in the scratch), lanes without
and with a second share of a species' production sum, and sizes of the call
down to one cell."""
import numpy as np
import pytest

from test_gpu_integrate import compare_cell_envelope, run_gpu, _say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


def _opts(precision):
    from paper_2312_13513_amd import chem
    o = chem.chem_default_opts()
    o.schedule = 1
    o.precision = precision
    return o


@pytest.mark.parametrize("K,R", [(5, 6), (15, 64), (16, 65), (23, 128), (24, 129), (35, 256), (35, 257), (36, 40),
                                 (47, 200), (48, 257), (63, 256), (63, 300)])
def test_wave_shapes_match_oracle(torch, tmp_path, oracle_lib, K, R):
    from chemgen.fields import cells4096
    from chemgen.mechanism import make_mechanism
    from paper_2312_13513_amd import chem
    p = tmp_path / "m.mech"
    m = make_mechanism(seed=20 + K, K=K, R=R, E=3 if K < 20 else 4)
    m.write(str(p))
    f = cells4096(m, n=19, seed=K + R)
    dt = 1e-7
    g = chem.Mechanism(str(p), 0)
    om = oracle_lib.OracleMech(str(p))
    tag = f"wave-K{K}-R{R}"
    _say(f"[{tag}] GPU run")
    got = run_gpu(torch, g, f.T, f.p, f.Y, dt, opts=_opts(0))
    ref = om.integrate(f.T, f.p, f.Y, dt)[:4]
    # every cell within four times the oracle's own spread under one- and
    # two-ulp changes of T and rtol, or the plain bars (1e-6 K, 1e-10)
    compare_cell_envelope(tag, om, f.T, f.p, f.Y, dt, *got, *ref, per_cell=False)
    # FP32 Jacobian and LU: the integration tolerance
    T32, Y32, s32, _ = run_gpu(torch, g, f.T, f.p, f.Y, dt, opts=_opts(1))
    assert np.all(s32 == 0) and np.abs(T32 - ref[0]).max() < 1e-3 and np.abs(Y32 - ref[1]).max() < 1e-6
    # a cell's result does not depend on the size of the call
    one = run_gpu(torch, g, f.T[:1], f.p[:1], np.ascontiguousarray(f.Y[:, :1]), dt, opts=_opts(0))
    assert np.array_equal(one[0], got[0][:1]) and np.array_equal(one[1], got[1][:, :1])
    g.close()
