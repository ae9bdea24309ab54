"""Which form the sums with weights on the fly take, and the sums by distance
bins at the edges of their blocks, bins and kernels, each case with the form it is
meant for (info["local_bins"])."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# A row sums n pairs x up to 48 lags of products whose weights carry a few ulps of
# the largest one (about 20 with the polynomial's and the sums' own rounding):
# relative to the largest sum of random histories 20 eps sqrt(48 n), 9e-13 for the
# largest n here (800).
TOL = 9e-13


@pytest.fixture(scope="module")
def wfp():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2507_07823_amd import wfp as w
    w.load_library()
    return w


def _problem(kind, M, dt, n, W=35, free=False):
    """M springs with about n neighbours each within W steps."""
    r = np.random.default_rng([len(kind), M])
    width = 2 * W * dt * M / n
    if kind == "slab":
        x = r.uniform(-2.0, -2.0 + width, M)
    elif kind == "seam":                  # both sides of the periodic seam, coincident springs
        x = np.where(np.arange(M) % 2 == 0, np.pi - 0.5 * width * r.random(M), -np.pi + 0.5 * width * r.random(M))
        x = np.minimum(x, np.pi - 1e-9)
        x[4] = x[2]
    else:                                 # springs exactly parts of a step apart
        x = -2.0 + dt * np.arange(M) / round(n / (2 * W))
    beta = 0.005 / dt ** 2 * width / M
    return dict(x=x, beta=np.full(M, beta), packets=np.array([[1.0, 0.0, 1.0, 20.0, 0.3]]), boundary=1 if free else 0,
                x_recv=np.array([-1.9, 0.25, 0.35]))


def _local(wfp, prob, dt, mode, **kw):
    import torch
    plan = wfp.Plan(prob, dt, local_mode=mode, **kw)
    i = plan.info
    g = torch.Generator(device="cuda").manual_seed(11)
    z = dict(device="cuda", dtype=torch.float64)
    plan.set_state(50, torch.randn(i["m_max"], i["M"], generator=g, **z), torch.zeros(i["W"], i["K"] + 1, 2, **z),
                   torch.zeros(i["K"] + 1, 2, **z), torch.zeros(i["K"] + 1, 2, **z))
    out = plan.local_part().cpu().numpy()
    plan.close()
    return i, out


# springs, neighbours, order -> by bins (1) or pair by pair (0)
@pytest.mark.parametrize("M,n,p,bins", [(7000, 160, 8, 1), (7000, 100, 8, 0), (2000, 130, 8, 0), (2000, 350, 8, 1),
                                        (256, 200, 8, 0), (20000, 140, 2, 0), (20000, 250, 2, 0), (20000, 450, 2, 1),
                                        (20000, 140, 4, 0), (20000, 300, 4, 1), (20000, 200, 6, 1), (2000, 200, 6, 0),
                                        (7000, 400, 10, 0)])
def test_form_of_weights_on_the_fly(wfp, M, n, p, bins):
    plan = wfp.Plan(_problem("slab", M, 2e-4, n), 2e-4, local_mode=2, p=p, K=4000)
    assert abs(plan.info["n_pairs"] / M / n - 1) < 0.25
    assert plan.info["local_mode"] == 2 and plan.info["local_bins"] == bins
    plan.close()


# springs, neighbours, order -> the library's choice
@pytest.mark.parametrize("M,n,p,mode", [(1000, 900, 8, 3), (3000, 560, 8, 3), (3000, 1450, 8, 2), (5000, 560, 4, 3),
                                        (10000, 560, 4, 3), (10000, 1000, 8, 2), (30000, 560, 8, 2), (30000, 400, 8, 3)])
def test_form_by_default(wfp, M, n, p, mode):
    prob = _problem("slab", M, 2e-4, n)
    plan = wfp.Plan(prob, 2e-4, p=p, K=4000)
    assert plan.info["local_mode"] == mode and plan.info["local_bins"] == (1 if mode == 2 else 0)
    plan.close()


# each layout (windows, quadratures, orders), and sizes at the edges of blocks (32
# sources) and of the reduction's rows (64); steps of four lags: 10, or 13 in the
# kernel that also takes cells with up to four edges
CASES = [
    dict(kind="slab", M=6016, n=300, dt=1e-3),
    dict(kind="slab", M=6017, n=300, dt=1e-3, free=True),
    dict(kind="slab", M=6047, n=500, dt=1e-3, p=2),
    dict(kind="slab", M=6049, n=400, dt=1e-3, p=4),
    dict(kind="slab", M=6080, n=250, dt=1e-3, p=6),
    dict(kind="slab", M=6081, n=300, dt=1e-3, W=36),              # 40 lags: the last of ten steps of four
    dict(kind="slab", M=6079, n=300, dt=1e-3, W=20),              # a steeper window, narrower bins
    dict(kind="seam", M=6003, n=300, dt=1e-3),
    dict(kind="seam", M=6001, n=800, dt=5e-3),                    # windows around much of the circle
    dict(kind="grid", M=6000, n=280, dt=1e-3),
    dict(kind="slab", M=6015, n=300, dt=1e-3, eps_window=1e-6),   # 13 steps: cells with several edges
    dict(kind="seam", M=6005, n=500, dt=1e-3, eps_window=1e-6, p=4),
    dict(kind="grid", M=6001, n=288, dt=1e-3, eps_window=1e-6, p=6),
    dict(kind="slab", M=6018, n=400, dt=1e-3, W=38, n_gl_local=28),   # 42 lags: 13 steps
    dict(kind="seam", M=6021, n=500, dt=1e-3, W=44, n_gl_local=20),   # 48
]


def _window(case):
    return case.get("W") or (18 if case.get("eps_window") else 35)


def _ids(case):
    return "-".join(f"{k}{v}" for k, v in case.items())


@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_bins_equal_stored_weights(wfp, case):
    kw = {k: case[k] for k in ("p", "W", "n_gl_local", "eps_window") if k in case}
    prob = _problem(case["kind"], case["M"], case["dt"], case["n"], _window(case), case.get("free", False))
    i, a = _local(wfp, prob, case["dt"], 2, **kw)
    assert i["local_mode"] == 2 and i["local_bins"] == 1
    j, b = _local(wfp, prob, case["dt"], 3, **kw)
    assert j["local_mode"] == 3 and j["local_bins"] == 0
    err = np.max(np.abs(a - b)) / np.max(np.abs(b))
    print(f"{case}: {err:.2e}", flush=True)
    assert err < TOL


@pytest.mark.parametrize("W,p", [(4, 8), (5, 8), (3, 6), (4, 6)])
def test_shortest_windows(wfp, W, p):
    """A window of p / 2 steps goes pair by pair, one step more by bins; both as with
    the weights stored."""
    kw = dict(p=p, W=W, eps_window=5e-3)
    prob = _problem("slab", 6020, 1e-3, 500, W)
    i, a = _local(wfp, prob, 1e-3, 2, **kw)
    assert i["local_mode"] == 2 and i["local_bins"] == (1 if W > p // 2 else 0)
    j, b = _local(wfp, prob, 1e-3, 3, **kw)
    err = np.max(np.abs(a - b)) / np.max(np.abs(b))
    print(f"W={W} p={p}: {err:.2e}", flush=True)
    assert err < TOL


@pytest.mark.parametrize("case", [CASES[3], CASES[7], CASES[10], CASES[13]], ids=_ids)
def test_bins_gradient_equals_stored_weights(wfp, case):
    """Both gradients (the derivative sums take blocks of 16 sources and two
    histories), against weights and derivatives stored once per pair."""
    import torch
    kw = {k: case[k] for k in ("p", "W", "n_gl_local", "eps_window") if k in case}
    prob = _problem(case["kind"], case["M"], case["dt"], case["n"], _window(case))
    n = 24
    e = torch.randn(n, 3, generator=torch.Generator().manual_seed(5), dtype=torch.float64).cuda()
    got = {}
    for mode in (2, 3):
        plan = wfp.Plan(prob, case["dt"], local_mode=mode, checkpoint_every=-20, **kw)
        assert plan.info["local_bins"] == (1 if mode == 2 else 0)
        plan.march(n)
        got[mode] = [v.cpu().numpy() for v in plan.gradient(e)]
        plan.close()
    for a, b in zip(got[2], got[3]):
        err = np.max(np.abs(a - b)) / np.max(np.abs(b))
        print(f"{case}: {err:.2e}", flush=True)
        # 24 levels of the sums above, forward and back
        assert err < 24 * TOL


# instances, springs, neighbours, parameters -> the library's choice: by bins only
# where they fit the batched kernel (768 bins, 40 lags, two edges a cell) and the
# launch is the shorter one
@pytest.mark.parametrize("n,M,nb,kw,mode", [(8, 1500, 450, dict(n_gl_local=40), 3), (8, 1500, 450, dict(eps_window=1e-6), 3),
                                            (1, 600, 580, {}, 3), (8, 3000, 480, {}, 2), (8, 3000, 480, dict(p=6), 3)])
def test_batch_form_by_default(wfp, n, M, nb, kw, mode):
    import torch
    dt, levels = 1e-3, 4
    W = 18 if "eps_window" in kw else 35
    probs = [dict(_problem("slab", M, dt, nb, W), x_recv=np.zeros(0)) for _ in range(n)]
    for i, p in enumerate(probs):
        p["x"] = p["x"] + 1e-4 * i
    b = wfp.Batch(probs, [dt] * n, **kw)
    infos = [b.plan(i).info for i in range(n)]
    assert all(i["n_pairs"] > 400 * M for i in infos)
    assert [i["local_mode"] for i in infos] == [mode] * n
    assert [i["local_bins"] for i in infos] == [1 if mode == 2 else 0] * n
    out = [torch.empty(M, dtype=torch.float64, device="cuda") for _ in range(n)]
    b.run(levels, out)
    b.close()
    for i in (0, n - 1):
        plan = wfp.Plan(probs[i], dt, local_mode=1, **kw)
        ref = plan.march(levels)[0][-1]
        plan.close()
        assert float((out[i] - ref).abs().max() / ref.abs().max()) < levels * TOL


# explicit weights on the fly: pair by pair where the bins do not fit or a few springs
# would wait for a whole round, without the tables of the bins
@pytest.mark.parametrize("n,M,nb,kw,bins", [(4, 1500, 200, dict(eps_window=1e-6), 0), (2, 300, 150, {}, 0),
                                            (8, 1500, 150, {}, 1)])
def test_batch_form_of_weights_on_the_fly(wfp, n, M, nb, kw, bins):
    probs = [dict(_problem("slab", M, 1e-3, nb, 18 if kw else 35), x_recv=np.zeros(0)) for _ in range(n)]
    b = wfp.Batch(probs, [1e-3] * n, local_mode=2, **kw)
    infos = [b.plan(i).info for i in range(n)]
    assert [(i["local_mode"], i["local_bins"]) for i in infos] == [(2, bins)] * n
    b.run(2)
    b.close()
