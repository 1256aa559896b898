"""The transport kernels with the species in groups of four, at the edges of
their group counts (5, 6, 9, 12, 16 groups: one species in the last group, a
full last group, whole groups of padding) and of their 16-cell tiles, against the
oracle with the bars of the other property tests (sums of K <= 64 positive
terms a few roundings apart: 1e-12 relative; diffusion plus 1e-15 / (1 - y)).
A cell's results are the same bits wherever it lies in the call."""
import numpy as np
import pytest

from test_gpu_thermo import _dev, _open, _state, _transport_check, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [17, 21, 24, 25, 33, 37, 48, 49, 61])
def test_group_edges(torch, tmp_path, K):  # noqa: F811
    from chemgen.transport import transport_fits
    mech, m, _ = _open(tmp_path, f"K{K}")
    fits = transport_fits(mech, 5)
    m.set_transport(*fits)
    n = 2049
    T, p, Y = _state(K, n, K)

    def call(a, b):
        out = [torch.full((b - a + 3,), float("nan"), dtype=torch.float64, device="cuda:0") for _ in range(2)]
        D = torch.full((K, b - a + 3), float("nan"), dtype=torch.float64, device="cuda:0")
        m.transport(_dev(torch, T[a:b]), _dev(torch, p[a:b]), _dev(torch, Y[:, a:b], b - a + 1), *out, D,
                    ncells=b - a)
        r = [v.cpu().numpy() for v in (*out, D)]
        assert all(np.isnan(v[..., b - a:]).all() for v in r), "written beyond ncells"
        return [v[..., :b - a] for v in r]

    whole = call(0, n)
    _transport_check(f"transport K{K}", mech, fits, T, p, Y, *whole)
    for a, b in ((0, 1), (5, 20), (1, 17), (n - 17, n)):
        for v, w in zip(call(a, b), whole):
            assert np.array_equal(v, w[..., a:b])
    m.close()
