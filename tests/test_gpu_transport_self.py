"""Diffusion coefficients of mixtures do not depend on the species' own
(self-diffusion) fits, which only a pure cell reads: with fits of zero on the
diagonal they are finite and have the bits of the calls with the real ones, at
the edges of the kernels' species bounds and group counts."""
import numpy as np
import pytest

from test_gpu_thermo import _dev, _open, _state, _transport_check, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [9, 14, 16, 17, 20, 21, 24, 25, 36, 61])
def test_mixtures_do_not_read_the_self_fits(torch, tmp_path, K):  # noqa: F811
    from chemgen.transport import transport_fits
    mech, m, _ = _open(tmp_path, f"K{K}")
    visc, cond, diff = transport_fits(mech, 5)
    n = 1025
    T, p, Y = (a[..., :n] for a in _state(K, n + (n + 60) // 50 + 1, K))   # without the pure cells
    none = diff.copy()
    none[np.arange(K), np.arange(K)] = 0.0
    out = []
    for fit in (diff, none):
        m.set_transport(visc, cond, fit)
        mu, lam = (torch.full((n,), float("nan"), dtype=torch.float64, device="cuda:0") for _ in range(2))
        D = torch.full((K, n), float("nan"), dtype=torch.float64, device="cuda:0")
        m.transport(_dev(torch, T), _dev(torch, p), _dev(torch, np.ascontiguousarray(Y)), mu, lam, D)
        out.append([v.cpu().numpy() for v in (mu, lam, D)])
    _transport_check(f"self fits K{K}", mech, (visc, cond, none), T, p, Y, *out[1])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    m.close()
