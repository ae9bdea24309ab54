"""The pair-once stored local sum at the edges of its blocks (8 or 16 rows) and
of the chunks of sources that it stages (128, 64 in the gradient pass), and the
history part at the edges of its lanes, columns and rows."""
import math

import numpy as np
import pytest

from oracle.history import mode_step, pq_tables, rotation
from oracle.rows import spectrum_direct

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wfp():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2507_07823_amd import wfp as w
    w.load_library()
    return w


def _problem(M, width, dt, seam=False, free=False):
    r = np.random.default_rng([5, M])
    x = r.uniform(0.2, 0.2 + width, M) - (2.7 if width > 4.0 else 0.0)
    if seam:
        x = np.where(np.arange(M) % 2 == 0, np.pi - width * r.random(M), -np.pi + width * r.random(M))
        x = np.minimum(x, np.pi - 1e-9)
    beta = 0.005 / dt ** 2 * width / M
    return dict(x=x, beta=np.full(M, beta), packets=np.array([[1.0, -2.0, 0.1, 0.0, 0.0]]), boundary=1 if free else 0,
                x_recv=np.array([0.15, 0.25, 0.35]))


def _state(plan, seed=11):
    import torch
    i = plan.info
    g = torch.Generator(device="cuda").manual_seed(seed)
    z = dict(device="cuda", dtype=torch.float64)
    s = dict(hist=torch.randn(i["m_max"], i["M"], generator=g, **z),
             ring=torch.randn(i["W"], i["K"] + 1, 2, generator=g, **z),
             alpha=torch.randn(i["K"] + 1, 2, generator=g, **z), dalpha=torch.randn(i["K"] + 1, 2, generator=g, **z))
    for k in ("ring", "alpha", "dalpha"):
        s[k][..., 0, 1] = 0.0
    return s


def _rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


# The two modes store the same weights to rounding and add a row's n pairs x 40
# lags in another order: relative to the largest sum of random histories
# 4 eps sqrt(40 n), 3e-13 for n = 4000.
LOCAL_TOL = 3e-13

PAIRS = [
    dict(M=1, width=0.1, dt=2e-3),
    dict(M=7, width=0.05, dt=2e-3),                       # one block, not full
    dict(M=17, width=0.01, dt=2e-3),
    dict(M=129, width=0.05, dt=2e-3, p=6),                # ranges of 128 and fewer: one chunk and one source more
    dict(M=300, width=0.06, dt=2e-3),                     # all in reach: ranges up to 300
    dict(M=2000, width=1.0, dt=2e-3, free=True),
    dict(M=501, width=0.05, dt=4e-3, seam=True),          # ranges that run on at source 0
    dict(M=8191, width=5.0, dt=1e-3),                     # the last size with 8 rows per block,
    dict(M=8192, width=5.0, dt=1e-3),                     # the first with 16
    dict(M=9001, width=2.0, dt=1e-3, p=4),
]


@pytest.mark.parametrize("case", PAIRS, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_pair_once_equals_per_pair(wfp, case):
    prob = _problem(case["M"], case["width"], case["dt"], case.get("seam"), case.get("free"))
    out = []
    for mode in (1, 3):
        plan = wfp.Plan(prob, case["dt"], p=case.get("p", 8), local_mode=mode)
        assert plan.info["local_mode"] == mode
        plan.set_state(50, **_state(plan))
        out.append(plan.march(3)[0])
        plan.close()
    assert _rel(out[1], out[0]) < LOCAL_TOL


@pytest.mark.parametrize("case", [PAIRS[i] for i in (1, 3, 4, 6)],
                         ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_pair_once_gradient_equals_per_pair(wfp, case):
    import torch
    prob = _problem(case["M"], case["width"], case["dt"], case.get("seam"))
    prob["packets"] = np.array([[1.0, 0.2, 0.2, 0.0, 0.0]])
    n = 12
    dJdu = torch.randn((n, 3), generator=torch.Generator().manual_seed(3), dtype=torch.float64).cuda()
    out = []
    for mode in (1, 3):
        plan = wfp.Plan(prob, case["dt"], p=case.get("p", 8), local_mode=mode, checkpoint_every=5)
        u = torch.empty((n, 3), dtype=torch.float64, device="cuda")
        plan.run(n, None, 1, u)
        out.append(plan.gradient(dJdu))
        plan.close()
    # the gradients sum n levels of such terms
    for a, b in zip(out[1], out[0]):
        assert _rel(a, b) < LOCAL_TOL * math.sqrt(n)


# A spectrum sums M spread terms that carry about 16 eps of rounding each,
# relative to the largest one of random densities 16 eps sqrt(M); a mode adds 40
# taps of such spectra.  K is a few hundred at most: the direct sum's phases k x
# carry k eps besides.
def _tol(M):
    return 16 * 2.2e-16 * math.sqrt(max(M, 40))


HISTORY = [
    dict(M=1, dt=0.0511),                                 # n1 = 5, n2 = 25
    dict(M=3, dt=0.08),                                   # K = 39
    dict(M=240, dt=0.02),                                 # 6 sources a cell on average: one lane,
    dict(M=241, dt=0.02),                                 # then two
    dict(M=700, dt=0.0101, free=True),                    # n1 = n2 = 25
    dict(M=6000, dt=0.02),                                # 32 lanes a cell
]


@pytest.mark.parametrize("case", HISTORY, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_history_step(wfp, case):
    """One level's spectrum and mode update against the direct sums."""
    M, dt = case["M"], case["dt"]
    prob = _problem(M, 2.0 if case.get("free") else 2.9, dt, free=case.get("free"))
    prob["x"] = prob["x"] - 1.3
    prob["x_recv"] = np.zeros(0)
    plan = wfp.Plan(prob, dt)
    i, s = plan.info, _state(plan)
    assert (50 % i["rbc_period"]) or not case.get("free")   # no boundary projection at this level
    plan.set_state(50, **s)
    plan.run(1)
    now = plan.get_state()
    plan.close()

    def cplx(t):
        t = t.cpu().numpy()
        return t[..., 0] + 1j * t[..., 1]
    K, W = i["K"], i["W"]
    S = spectrum_direct(prob["x"], s["hist"][0].cpu().numpy(), K)
    ring = np.concatenate([S[None], cplx(s["ring"])[:-1]])
    P, Q = pq_tables(K, dt, W, W * dt, math.log(1e12))
    al, da = mode_step(cplx(s["alpha"]), cplx(s["dalpha"]), ring, P, Q, rotation(K, dt), dt)
    for got, want in ((now["ring"][0], S), (now["alpha"], al), (now["dalpha"], da)):
        assert np.abs(cplx(got) - want).max() <= _tol(M) * np.abs(want).max()


# Dense coupling solved by global sweeps, 16 or 64 rows a block: the densities
# satisfy (I + S) sigma = b, so a march equals one whose springs' order and
# whose tiles differ only to the sums' rounding and the sweeps' 1e-18: with n
# nearby springs a row 4 eps sqrt(n), 4e-14 for the 2000 here, on top of the
# local sums.
SWEEPS = [
    dict(M=700, width=0.002, dt=2e-3),                    # all coupled; the last block has 12 rows of 16
    dict(M=2049, width=0.01, dt=2e-3, seam=True),         # runs across source 0, one row in the last 64
    dict(M=40001, width=0.4, dt=2e-3),                    # 64 rows a block, one row in the last
]


@pytest.mark.parametrize("case", SWEEPS, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_global_sweeps_solve_the_level(wfp, case):
    """The solved level against the residual of its own equation, the coupling
    by the oracle's weights."""
    from oracle.local import local_weights
    M, dt = case["M"], case["dt"]
    prob = _problem(M, case["width"], dt, case.get("seam"))
    prob["x_recv"] = np.zeros(0)
    out = []
    for it in (0, 14):
        plan = wfp.Plan(prob, dt, local_mode=2, solve_iters=it)
        i = plan.info
        assert i["solve_mode"] == 1
        plan.set_state(50, **_state(plan))
        out.append(plan.march(1)[0][0].cpu().numpy())
        plan.close()
    # more sweeps change nothing
    assert np.abs(out[1] - out[0]).max() <= LOCAL_TOL * np.abs(out[0]).max()
    # one sweep from zero is the right-hand side over the diagonal
    plan = wfp.Plan(prob, dt, local_mode=2, solve_iters=1)
    plan.set_state(50, **_state(plan))
    x1 = plan.march(1)[0][0].cpu().numpy()
    plan.close()
    order = np.argsort(np.mod(prob["x"], 2 * np.pi) if case.get("seam") else prob["x"], kind="stable")
    x, beta, sig, x1 = (v[order] for v in (np.mod(prob["x"], 2 * np.pi) if case.get("seam") else prob["x"],
                                           prob["beta"], out[0], x1))
    prm = dict(W=i["W"], p=8, delta=i["W"] * dt, b=math.log(1e12), n_gl=i["W"])
    s0 = 0.5 * beta * local_weights(np.zeros(1), dt, **prm)[0, 0]
    rows = np.unique(np.r_[0, 1, M // 2, M - 2, M - 1, np.random.default_rng(1).integers(0, M, 20)])
    for j in rows:
        near = np.flatnonzero(np.abs(x - x[j]) < dt)
        q = 0.5 * beta[j] * local_weights(np.abs(x[near] - x[j]), dt, **prm)[:, 0]
        lhs = sig[j] + q @ sig[near]
        rhs = x1[j] * (1.0 + s0[j])
        assert abs(lhs - rhs) <= LOCAL_TOL * np.abs(out[0]).max()
