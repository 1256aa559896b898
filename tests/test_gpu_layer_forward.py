"""The layer kernel of wide networks against the general product, bit for bit:
the same rows in a call large enough for the layer kernel and in small pieces
that take the general one, at row counts around its 128-row blocks and unit
counts whose last 256-unit block has one, two, three or four waves."""
import numpy as np
import pytest

from test_gpu_surrogate import _say, mechs, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h", [(64, 128, 192), (1600, 800, 400), (256, 320, 64)])
@pytest.mark.parametrize("rows", [1024, 1151, 1153, 2177])
def test_layer_kernel_equals_general_product(torch, mechs, h, rows):  # noqa: F811
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
    for a in range(0, rows, 16):   # one row block: 9 to 57 tiles a layer, below the layer kernel's 64
        n = min(16, rows - a)
        o = torch.zeros((n, s.nout_pad), device="cuda:0")
        s.forward(X[a:a + n].contiguous(), o)
        ref[a:a + n] = o
    assert np.isfinite(out.cpu().numpy()).all()
    assert torch.equal(out, ref)
    s.close()
