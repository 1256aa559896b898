"""The fused training kernels at the edges of their shapes: batches around the
16-row blocks, the 32-row steps and the row ranges of the bias sums, widths
from 64 to 512, 9 and 35 species, a shuffled order with a last short batch;
gradients against the FP64 oracle, and a training run against single gradient
and Adam steps, bit for bit."""
import numpy as np
import pytest

from test_gpu_surrogate import _dev, _surr, _synthetic_norm, _say, mechs, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,K,h", [("M9", 9, (64, 64, 64)), ("M35", 35, (512, 64, 512)), ("M35", 35, (128, 512, 192))])
def test_gradient_at_block_edges(torch, mechs, name, K, h):  # noqa: F811
    from chemgen.surrogate_data import split_params
    from oracle import surrogate as S
    from paper_2312_13513_amd import chem
    s, dims, flat = _surr(chem, mechs[name], K, h=h, seed=41)
    rng = np.random.default_rng(42)
    n = 2049
    x = S.to_bf16(rng.normal(0, 1, (n, K + 2)).astype(np.float32))
    Xb = np.zeros((n, 64), dtype=np.uint16)
    Xb[:, :K + 2] = S.bf16_bits(x)
    tgt = rng.normal(0, 1, (n, K)).astype(np.float32)
    X = torch.tensor(Xb.view(np.int16), device="cuda:0")
    Yt = _dev(torch, tgt, torch.float32)
    params_bf = [(S.to_bf16(W.astype(np.float32)), b) for W, b in split_params(flat, dims)]
    for rows in (1, 15, 16, 17, 32, 33, 511, 512, 513, 2048, 2049):
        loss = s.grad(X[:rows].contiguous(), Yt[:rows].contiguous())
        gg = split_params(s.get_grads(), dims)
        out, cache = S.forward(params_bf, x[:rows])
        t = tgt[:rows].astype(np.float64)
        grads = S.backward(params_bf, cache, out, t)
        worst = 0.0
        for (gW, gb), (rW, rb) in zip(gg, grads):
            for a, r in ((gW, rW), (gb, rb)):
                worst = max(worst, np.linalg.norm(a - r) / np.linalg.norm(r))
        _say(f"[grad {name} {h} rows {rows}] loss {loss:.6e}, worst rel-L2 of a layer {worst:.3e}")
        # activations and errors are rounded to BF16 (unit roundoff 2^-8) in three layers each way
        assert worst <= 2e-2 and abs(loss - S.mse_loss(out, t)) <= 1e-2 * S.mse_loss(out, t)
    s.close()


@pytest.mark.parametrize("n,batch", [(1000, 257), (640, 512), (48, 64)])
def test_training_equals_single_steps(torch, mechs, n, batch):  # noqa: F811
    from chemgen.surrogate_data import epoch_orders, flame_like_states
    from chemgen.mechanism import standard_mechanism
    from paper_2312_13513_amd import chem
    K = 35
    T, p, Y = flame_like_states(standard_mechanism("M35"), n, 5)
    Yn = Y * np.exp(0.01 * np.random.default_rng(6).normal(size=Y.shape))
    dT, dp, dY, dYn = (_dev(torch, a, torch.float64) for a in (T, p, Y, Yn))
    nets = []
    for _ in range(2):
        s, dims, flat = _surr(chem, mechs["M35"], K, seed=51)
        s.fit_norm(dT, dp, dY, dYn, 1e-5)
        nets.append(s)
    order = epoch_orders(n, 2, 7)
    nets[0].train(dT, dp, dY, dYn, 2, batch, lr0=1e-3, lr1=1e-5, order=torch.tensor(order, device="cuda:0"))
    a = nets[1]
    norm = a.get_norm()
    X = torch.zeros((n, 64), dtype=torch.int16, device="cuda:0")
    a.encode(dT, dp, dY, X)
    mu, sg = norm[2 * (K + 2):2 * (K + 2) + K], norm[2 * (K + 2) + K:-1]
    ok = sg >= 1e-12
    yt = np.where(ok, ((Yn - Y).T - mu) / np.where(ok, sg, 1.0), 0.0).astype(np.float32)
    Yt = torch.tensor(yt, device="cuda:0")
    per = -(-n // batch)
    step = 0
    for ep in range(2):
        for b in range(per):
            idx = torch.tensor(order[ep * n + b * batch:min(ep * n + (b + 1) * batch, (ep + 1) * n)].astype(np.int64), device="cuda:0")
            a.grad(X[idx].contiguous(), Yt[idx].contiguous())
            a.adam(1e-5 + 0.5 * (1e-3 - 1e-5) * (1.0 + np.cos(np.pi * step / (2 * per))))
            step += 1
    assert np.array_equal(nets[0].get_params(), a.get_params())
    for s in nets:
        s.close()
