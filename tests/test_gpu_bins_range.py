"""The sum by distance bins where a block of 32 sources reaches across the box
and the step is so short that a distance in lookup cells exceeds an int."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# as for the other sums by bins: 20 eps sqrt(40 n) of the largest sum, n = 530
TOL = 7e-13


@pytest.fixture(scope="module")
def wfp():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2507_07823_amd import wfp as w
    w.load_library()
    return w


@pytest.mark.parametrize("free", [False, True])
@pytest.mark.parametrize("p,dt", [(8, 2e-7), (2, 5e-7)])
def test_two_clumps_far_apart(wfp, p, dt, free):
    """Sources 2976 .. 3007 lie in both clumps, 1.8 apart: 9e6 and 3.6e6 steps, more
    than 2^31 lookup cells of the lowest bins.  They do not see each other."""
    import torch
    r = np.random.default_rng(7)
    x = np.concatenate([-1.0 + 400 * dt * r.random(3000), 0.8 + 400 * dt * r.random(3000)])
    M = x.size
    beta = np.full(M, 0.005 / dt ** 2 * 400 * dt / 3000)
    prob = dict(x=x, beta=beta, packets=np.array([[1.0, -2.0, 0.1, 0.0, 0.0]]), boundary=1 if free else 0)
    out = []
    for mode in (2, 3):
        plan = wfp.Plan(prob, dt, local_mode=mode, p=p, K=2000)
        i = plan.info
        assert i["local_mode"] == mode and i["local_bins"] == (1 if mode == 2 else 0)
        g = torch.Generator(device="cuda").manual_seed(11)
        z = dict(device="cuda", dtype=torch.float64)
        plan.set_state(50, torch.randn(i["m_max"], M, generator=g, **z), torch.zeros(i["W"], 2001, 2, **z),
                       torch.zeros(2001, 2, **z), torch.zeros(2001, 2, **z))
        out.append(plan.local_part().cpu().numpy())
        plan.close()
    err = np.max(np.abs(out[0] - out[1])) / np.max(np.abs(out[1]))
    print(f"p={p} dt={dt}: {err:.2e}", flush=True)
    assert err < TOL
