"""The solve's global sweeps in their forms (a wavefront per row, and the diagonals
with 16 or 64 rows a block): a dense cluster's densities do not depend on how many
lone springs stand elsewhere, while the form does."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wfp():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2507_07823_amd import wfp as w
    w.load_library()
    return w


# a cluster (ragged runs where it spans three steps), and the lone springs beside it:
# alone a wavefront per row (up to 2.5e6 entries) or 16 rows a block, with them 64
@pytest.mark.parametrize("n,span,seam,more", [(701, 0.9, False, 9000), (1501, 3.0, False, 9000), (1601, 3.0, True, 9000),
                                              (1701, 0.9, False, 9000), (2401, 3.0, True, 11000)])
def test_forms_of_the_sweeps(wfp, n, span, seam, more):
    """The first level solves (I + S) sigma = g, without a past.  A row adds n products;
    rounding is amplified by at most 1 / (1 - rho): 4 eps sqrt(n) / (1 - rho)."""
    dt = 1e-4
    r = np.random.default_rng(n)
    centre = np.pi if seam else 1.0
    x = centre + span * dt * (r.random(n) - 0.5)
    x = np.where(x >= np.pi, x - 2 * np.pi, x)
    beta = r.uniform(0.5, 1.0, n) * (0.5 / (dt * n))
    got = []
    for lone in (0, more):
        y = -2.5 + 2.5e-4 * np.arange(lone)
        prob = dict(x=np.concatenate([x, y]), beta=np.concatenate([beta, np.full(lone, 1e-3)]),
                    packets=np.array([[1.0, centre if not seam else 3.0, 0.5, 3.0, 0.3]]), boundary=0)
        plan = wfp.Plan(prob, dt, local_mode=2, K=1000)
        i = plan.info
        assert i["solve_mode"] == 1 and i["solve_contraction"] < 0.8
        got.append(plan.march(1)[0][0].cpu().numpy()[:n])
        tol = 4 * 2.2e-16 * np.sqrt(n) / (1 - i["solve_contraction"])
        plan.close()
    err = np.max(np.abs(got[1] - got[0])) / np.max(np.abs(got[0]))
    print(f"n={n} span={span} seam={seam}: {err:.2e} of {tol:.2e}", flush=True)
    assert err < tol
