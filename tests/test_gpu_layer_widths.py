"""The layer kernel of wide networks against the general product, bit for bit,
where its last 256-unit block has one to four active waves and around the sizes
at which a layer moves from one to the other: a call's rows against the same
rows in small pieces, which take the general product."""
import numpy as np
import pytest

from test_gpu_surrogate import mechs, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,rows", [((320, 384, 128), 1025), ((320, 384, 128), 1281), ((448, 64, 512), 1153),
                                    ((64, 128, 256), 4097), ((128, 64, 128), 8200), ((192, 448, 64), 6300)])
def test_call_equals_its_pieces(torch, mechs, h, rows):  # noqa: F811
    from chemgen.surrogate_data import init_species_params
    from paper_2312_13513_amd import chem
    K = 9
    s = chem.Surrogate(mechs["M9"], *h, per_species=True)
    s.set_params(init_species_params(K, h, 3))
    g = torch.Generator(device="cuda:0").manual_seed(rows)
    x = torch.randn((rows, 64), generator=g, device="cuda:0")
    x[:, K + 2:] = 0
    X = x.bfloat16().view(torch.int16).contiguous()
    out = torch.zeros((rows, s.nout_pad), device="cuda:0")
    s.forward(X, out)
    ref = torch.zeros_like(out)
    for a in range(0, rows, 64):   # one row block: below the layer kernel's 64 blocks
        n = min(64, rows - a)
        o = torch.zeros((n, s.nout_pad), device="cuda:0")
        s.forward(X[a:a + n].contiguous(), o)
        ref[a:a + n] = o
    assert np.isfinite(out.cpu().numpy()).all()
    assert torch.equal(out, ref)
    s.close()
