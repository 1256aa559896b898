"""Encoding and decode with 16 cells per wave, at the edges of their species
bounds (full and one-over) and of their 16-cell tiles, against the oracle with the bars
of the other surrogate tests (at most one BF16 code off by one; the accept mask
equal, T within 1e-8 K, Y within 1e-14).  A cell's results are the same bits wherever
it lies in the call."""
import numpy as np
import pytest

from test_gpu_surrogate import _synthetic_norm
from test_gpu_thermo import _dev, _open, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [10, 11, 12, 13, 22, 24, 25, 36, 38, 39, 48, 49, 62])
def test_species_and_tile_edges(torch, tmp_path, oracle_lib, K):  # noqa: F811
    from oracle import surrogate as S
    from paper_2312_13513_amd import chem
    mech, m, path = _open(tmp_path, f"K{K}")
    om = oracle_lib.OracleMech(path)
    rng = np.random.default_rng(K)
    n = 81
    T = rng.uniform(700.0, 2500.0, n)
    p = rng.uniform(0.5, 4.0, n) * 101325.0
    Y = rng.dirichlet(np.full(K, 0.6), n).T.copy()
    W = mech.molar_masses()
    norm = _synthetic_norm(T, p, Y, K, rng)
    norm[2 * K + 4:3 * K + 4] = 0.0
    mu_y, sig_y = norm[2 * K + 4:3 * K + 4], norm[3 * K + 4:4 * K + 4]
    sig_y[:] = 1e-4
    yhat = rng.normal(0, 1, (n, K))          # breaks the elements: rejected
    for i in range(0, n, 2):                 # along a reaction: accepted unless a fraction goes negative
        r = mech.reactions[int(rng.integers(len(mech.reactions)))]
        nu = np.zeros(K)
        for side, sign in ((r[0], -1.0), (r[1], 1.0)):
            for k, c in side:
                nu[k] += sign * c
        yhat[i] = 0.1 * nu * W / max(np.max(np.abs(nu * W)), 1e-300)
    yhat[::8] = 0.0
    yhat[3, K - 1] = np.nan
    yhat[6, 0] = np.inf
    s = chem.Surrogate(m, 64, 64, 64)
    s.set_norm(norm)
    out = np.zeros((n, s.nout_pad), dtype=np.float32)
    out[:, :K] = yhat

    def call(a, b):
        ld = b - a + 3
        Td, pd, Yd = _dev(torch, T[a:b]), _dev(torch, p[a:b]), _dev(torch, Y[:, a:b], ld)
        X = torch.full((b - a + 1, 64), 77, dtype=torch.int16, device="cuda:0")
        s.encode(Td, pd, Yd, X)
        mask = torch.full((b - a + 1,), 77, dtype=torch.int32, device="cuda:0")
        s.apply(Td, pd, Yd, _dev(torch, out[a:b], dtype=torch.float32), mask=mask)
        X, mask = X.cpu().numpy(), mask.cpu().numpy()
        assert np.all(X[b - a:] == 77) and mask[b - a] == 77, "written beyond ncells"
        assert np.all(np.isnan(Yd.cpu().numpy()[:, b - a:]))
        return X[:b - a].view(np.uint16), Td.cpu().numpy(), Yd.cpu().numpy()[:, :b - a], mask[:b - a]

    X, Tg, Yg, mk = whole = call(0, n)
    ref = np.zeros_like(X)
    ref[:, :K + 2] = S.bf16_bits(S.encode_cells(S.unpack_norm(norm, K), T, p, Y))
    off = np.abs(X.astype(np.int32) - ref.astype(np.int32))
    assert (off > 0).sum() <= 1 and off.max() <= 1
    ok = np.zeros(n, dtype=bool)
    for i in range(n):
        ok[i], Tn, Yn = S.apply_cell(om, mech.counts, W, T[i], Y[:, i], out[i, :K].astype(np.float64), mu_y, sig_y)
        assert abs(Tg[i] - Tn) < 1e-8 and np.max(np.abs(Yg[:, i] - Yn)) < 1e-14
    assert np.array_equal(mk == 0, ok) and 0 < ok.sum() < n
    for a, b in ((0, 1), (5, 20), (1, 17), (n - 17, n)):
        for v, w in zip(call(a, b), whole):
            assert np.array_equal(v, w[..., a:b] if w.ndim == 2 and w.shape[0] == K else w[a:b])
    s.close()
    m.close()
