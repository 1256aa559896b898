"""Captured inference calls of several passes with a compiled-in mechanism,
whose integrator needs workspace for every pass in flight: whatever sized it
(an eager call of one pass, of a full and a shorter one, of wider passes, or
chem_surrogate_reserve alone), the captured call is accepted and every replay
gives the bits of an eager one."""
import numpy as np
import pytest

from test_gpu_graph import _dev, _replay_check, torch  # noqa: F401

pytestmark = pytest.mark.gpu

PASS = 1024


def _surrogate(chem, mech, K, norm):
    from chemgen.surrogate_data import init_params, network_dims
    s = chem.Surrogate(mech, 64, 64, 64)
    s.set_params(init_params(network_dims(K, 64, 64, 64), 3))
    s.set_norm(norm)
    return s


@pytest.mark.parametrize("sized_by", ["one pass", "full and short pass", "wider pass", "reserve"])
def test_captured_passes(torch, mech_dir, sized_by):  # noqa: F811
    from chemgen.fields import cells4096
    from chemgen.mechanism import read_mechanism
    from oracle import surrogate as S
    from paper_2312_13513_amd import chem
    mpy = read_mechanism(str(mech_dir / "M9.mech"))
    f = cells4096(mpy, n=2 * PASS + (0 if sized_by != "reserve" else PASS // 2), seed=9)
    K = mpy.K
    mech = chem.Mechanism(str(mech_dir / "M9.mech"), 0)
    raw = S.features(f.T, f.p, f.Y)
    rng = np.random.default_rng(4)
    sig = raw.std(0)
    norm = np.concatenate([raw.mean(0), sig, np.zeros(K), rng.uniform(1e-10, 1e-9, K), [f.dt]])
    checks = chem.chem_surrogate_default_checks()
    checks.T_in_max = float(np.median(f.T))     # about half of each pass goes to the integrator
    T0, p, Y0 = _dev(torch, f.T), _dev(torch, f.p), _dev(torch, f.Y)
    T, Y = T0.clone(), Y0.clone()
    mask = torch.zeros(f.n, dtype=torch.int32, device="cuda:0")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    # the reference: an eager call of its own handle
    one = _surrogate(chem, mech, K, norm)
    one.infer(T, p, Y, f.dt, checks=checks, mask=mask, fallback_count=cnt)
    torch.cuda.synchronize()
    ref = (T.clone(), Y.clone(), mask.clone(), cnt.clone())
    assert 0 < int(mask[:PASS].sum()) < PASS and 0 < int(mask[PASS:].sum()) < f.n - PASS
    # the captured handle
    surr = _surrogate(chem, mech, K, norm)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    surr.set_pass_rows(PASS)

    def eager_call(n):
        surr.infer(T0[:n].clone(), p[:n], Y0[:, :n].clone(memory_format=torch.contiguous_format), f.dt, checks=checks,
                   stream=s)

    with torch.cuda.stream(s):
        if sized_by == "one pass":
            eager_call(PASS)
            surr.reserve(f.n)
        elif sized_by == "full and short pass":
            eager_call(PASS + PASS // 2)
            surr.reserve(f.n)
        elif sized_by == "wider pass":
            surr.set_pass_rows(0)
            eager_call(f.n)          # one pass: one side stream's workspace, as large as all cells
            surr.set_pass_rows(PASS)
        else:
            surr.reserve(f.n)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            T.copy_(T0)
            Y.copy_(Y0)
            surr.infer(T, p, Y, f.dt, checks=checks, mask=mask, fallback_count=cnt, stream=s)
    torch.cuda.synchronize()

    def eager():
        T.fill_(0.0)
        Y.fill_(0.0)
        mask.fill_(7)
        cnt.fill_(-3)
        one.infer(T0.clone(), p, Y0.clone(), f.dt, checks=checks)

    _replay_check(torch, g, (T, Y, mask, cnt), ref, eager)
    del g
    surr.close()
    one.close()
    mech.close()


def test_refused_call_joins_its_side_streams(torch, mech_dir):  # noqa: F811
    """A call that the integrator refuses (a negative tolerance) after work went to
    a side stream: the side stream is joined, so the capture it stood in can be
    ended, and the handle serves the next call."""
    from chemgen.fields import cells4096
    from chemgen.mechanism import read_mechanism
    from oracle import surrogate as S
    from paper_2312_13513_amd import chem
    mpy = read_mechanism(str(mech_dir / "M9.mech"))
    f = cells4096(mpy, n=PASS + 100, seed=9)
    mech = chem.Mechanism(str(mech_dir / "M9.mech"), 0)
    raw = S.features(f.T, f.p, f.Y)
    norm = np.concatenate([raw.mean(0), raw.std(0), np.zeros(mpy.K), np.full(mpy.K, 1e-9), [f.dt]])
    surr = _surrogate(chem, mech, mpy.K, norm)
    surr.set_pass_rows(PASS)
    p = _dev(torch, f.p)
    out = []
    for _ in range(2):
        T, Y = _dev(torch, f.T), _dev(torch, f.Y)
        surr.infer(T, p, Y, f.dt)
        torch.cuda.synchronize()
        out.append((T, Y))
        if len(out) == 1:
            opts = chem.chem_default_opts()
            opts.rtol = -1.0
            Tc, Yc = _dev(torch, f.T), _dev(torch, f.Y)
            s = torch.cuda.Stream()
            s.wait_stream(torch.cuda.current_stream())
            g = torch.cuda.CUDAGraph()
            with torch.cuda.stream(s), pytest.raises(chem.ChemError, match="rtol"):
                with torch.cuda.graph(g, stream=s):
                    surr.infer(Tc, p, Yc, f.dt, opts=opts, stream=s)
            torch.cuda.synchronize()
            del g
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    surr.close()
    mech.close()
