"""What the sums by distance bins add to the first gradient of a plan."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_first_gradient_costs_little_more_than_a_later_one():
    """M = 2e4, 240 neighbours: the derivatives' table and the 1250 blocks' windows
    are laid out in the first gradient.  Row by row copies of the windows made that
    11 ms; pair by pair, with three buffers to allocate, it is 3.7.  The best of
    three fresh plans has to stay below 6."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2507_07823_amd import wfp
    M, n, dt = 20_000, 12, 8.6e-4
    r = np.random.default_rng(3)
    prob = dict(x=r.uniform(-2.5, 2.5, M), beta=np.full(M, 0.005 / dt ** 2 * 5.0 / M),
                packets=np.array([[1.0, -2.0, 0.3, 20.0, 0.3]]), x_recv=np.linspace(-2.4, 2.0, 16))
    e = torch.randn(n, 16, generator=torch.Generator().manual_seed(5), dtype=torch.float64).cuda()

    def timed(plan):
        torch.cuda.synchronize()
        t = time.perf_counter()
        plan.gradient(e)
        torch.cuda.synchronize()
        return 1e3 * (time.perf_counter() - t)

    extra = []
    for _ in range(3):
        plan = wfp.Plan(prob, dt, local_mode=2, checkpoint_every=-250)
        assert plan.info["n_pairs"] > 230 * M
        plan.march(n)
        first = timed(plan)
        extra.append(first - min(timed(plan) for _ in range(3)))
        plan.close()
    print("first gradient, more than a later one, ms:", [round(v, 2) for v in extra], flush=True)
    assert min(extra) < 6.0
