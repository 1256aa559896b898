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


def test_captured_layers_follow_the_weights(torch, mechs):  # noqa: F811
    """A captured forward pass uses the weights of its replay, and capturing one with
    new weights leaves the eager pass right: both against a network that had the
    weights from the start, bit for bit, over several replays with eager work between."""
    from chemgen.surrogate_data import init_species_params
    from paper_2312_13513_amd import chem
    h, rows = (256, 320, 64), 1153
    par = [init_species_params(9, h, seed) for seed in (3, 4)]
    g = torch.Generator(device="cuda:0").manual_seed(1)
    X = torch.randn((rows, 64), generator=g, device="cuda:0").bfloat16().view(torch.int16).contiguous()
    refs = []
    for v in par:
        s = chem.Surrogate(mechs["M9"], *h, per_species=True)
        s.set_params(v)
        refs.append(torch.zeros((rows, s.nout_pad), device="cuda:0"))
        s.forward(X, refs[-1])
        torch.cuda.synchronize()
        s.close()
    assert not torch.equal(*refs)
    s = chem.Surrogate(mechs["M9"], *h, per_species=True)
    s.set_params(par[0])
    eager = torch.zeros_like(refs[0])
    s.forward(X, eager)              # sizes the workspace
    side = torch.cuda.Stream()
    for cur in (0, 1, 0):
        torch.cuda.synchronize()
        s.set_params(par[cur])
        out = torch.zeros_like(eager)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                s.forward(X, out, stream=side)
        torch.cuda.synchronize()
        s.forward(X, eager)          # before any replay
        torch.cuda.synchronize()
        assert torch.equal(eager, refs[cur])
        for new in (cur, 1 - cur, cur):
            s.set_params(par[new])
            out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, refs[new])
            s.forward(X, eager)
            torch.cuda.synchronize()
            assert torch.equal(eager, refs[new])
    s.close()
