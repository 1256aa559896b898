"""The wave-per-cell integrator with its reaction scratch in global memory
(from 878 elementary reactions, from 769 where some are pressure dependent),
against the oracle."""
import numpy as np
import pytest

from test_gpu_integrate import compare_cell_envelope, run_gpu, _say
from test_gpu_wave_shapes import _opts, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,R,pdep", [(40, 878, False), (45, 1030, False), (60, 900, False), (36, 769, True),
                                      (41, 890, True), (40, 1023, True), (63, 1100, True)])
def test_global_scratch_matches_oracle(torch, tmp_path, oracle_lib, K, R, pdep):  # noqa: F811
    from chemgen.fields import cells4096
    from chemgen.mechanism import make_mechanism, make_real_like_mechanism
    from paper_2312_13513_amd import chem
    assert R >= (769 if pdep else 878)   # the limits that test_wave_scratch.py holds the library to
    m = make_real_like_mechanism(seed=70 + K, K=K, R=R, E=4, n_third=30, n_lind=9, n_troe=12, n_dup=6,
                                 n_irrev=5) if pdep else make_mechanism(seed=70 + K, K=K, R=R, E=4)
    p = tmp_path / "m.mech"
    m.write(str(p))
    f = cells4096(m, n=19, seed=K + R)
    dt = 1e-8
    g = chem.Mechanism(str(p), 0)
    om = oracle_lib.OracleMech(str(p))
    tag = f"global-K{K}-R{R}-{'pdep' if pdep else 'elem'}"
    _say(f"[{tag}] GPU run")
    got = run_gpu(torch, g, f.T, f.p, f.Y, dt, opts=_opts(0))
    ref = om.integrate(f.T, f.p, f.Y, dt)[:4]
    # every cell within four times the oracle's own spread under one- and
    # two-ulp changes of T and rtol, or the plain bars (1e-6 K, 1e-10)
    compare_cell_envelope(tag, om, f.T, f.p, f.Y, dt, *got, *ref, per_cell=False)
    # FP32 Jacobian and LU: the integration tolerance
    T32, Y32, s32, _ = run_gpu(torch, g, f.T, f.p, f.Y, dt, opts=_opts(1))
    assert np.all(s32 == 0) and np.abs(T32 - ref[0]).max() < 1e-3 and np.abs(Y32 - ref[1]).max() < 1e-6
    # repeated and alone: a cell's bits depend neither on its slice nor on the call's size
    again = run_gpu(torch, g, f.T, f.p, f.Y, dt, opts=_opts(0))
    one = run_gpu(torch, g, f.T[:1], f.p[:1], np.ascontiguousarray(f.Y[:, :1]), dt, opts=_opts(0))
    for a, b, c in zip(got[:2], again[:2], one[:2]):
        assert np.array_equal(a, b) and np.array_equal(a[..., :1], c)
    g.close()
