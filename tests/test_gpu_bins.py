"""Local sums by distance bins (local_mode 2 from 112 neighbours per spring on):
the same sums as with the weights stored, at the edges of the kernel's blocks
(32 sources, 64 springs per reduce), of its bins and of its lag steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# A row sums n pairs x 40 lags of products whose weights carry a few ulps of
# the largest one (about 20 with the polynomial's and the sums' own rounding):
# relative to the largest sum of random histories, 20 eps sqrt(40 n), 6e-13 for
# the largest n here.
TOL = 6e-13


@pytest.fixture(scope="module")
def wfp():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2507_07823_amd import wfp as w
    w.load_library()
    return w


def _problem(case, seed=3):
    r = np.random.default_rng([seed, len(case["kind"]), case["M"]])
    M = case["M"]
    if case["kind"] == "slab":
        x = r.uniform(0.2, 0.2 + case["width"], M)
    elif case["kind"] == "seam":          # both sides of the periodic seam, coincident springs
        x = np.where(np.arange(M) % 2 == 0, np.pi - case["width"] * r.random(M),
                     -np.pi + case["width"] * r.random(M))
        x = np.minimum(x, np.pi - 1e-9)
        x[4] = x[2]
    else:                                 # springs exactly dt and several bins apart
        x = 0.1 + case["dt"] * np.arange(M) / 4.0
    # springs as stiff as the march stays stable with (dt sqrt(rho beta) = 0.07)
    beta = 0.005 / case["dt"] ** 2 * np.ptp(np.where(x < 0, x + 2 * np.pi, x)) / M
    return dict(x=x, beta=np.full(M, beta), packets=np.array([[1.0, -2.0, 0.1, 0.0, 0.0]]),
                boundary=1 if case.get("free") else 0, x_recv=np.array([0.15, 0.25, 0.35]))


def _histories(plan, seed=11):
    import torch
    i = plan.info
    g = torch.Generator(device="cuda").manual_seed(seed)
    z = dict(device="cuda", dtype=torch.float64)
    return dict(hist=torch.randn(i["m_max"], i["M"], generator=g, **z), ring=torch.zeros(i["W"], i["K"] + 1, 2, **z),
                alpha=torch.zeros(i["K"] + 1, 2, **z), dalpha=torch.zeros(i["K"] + 1, 2, **z))


CASES = [
    dict(kind="slab", M=113, width=0.01, dt=1e-3),                 # all within reach, ragged blocks
    dict(kind="slab", M=256, width=0.02, dt=1e-3, p=2),
    dict(kind="slab", M=1025, width=0.3, dt=4e-3, p=4),
    dict(kind="slab", M=1087, width=0.2, dt=2e-3, p=6, free=True),
    dict(kind="slab", M=700, width=0.1, dt=2e-3, W=36),            # 40 lags: the last of ten steps of four
    dict(kind="slab", M=700, width=0.1, dt=2e-3, W=37),            # 41: thirteen steps
    dict(kind="slab", M=700, width=0.1, dt=2e-3, W=20),            # a steeper window, narrower bins
    dict(kind="seam", M=603, width=0.05, dt=4e-3),
    dict(kind="seam", M=601, width=0.6, dt=0.08, n_gl_local=40),   # windows around most of the circle
    dict(kind="grid", M=900, dt=2e-3),
    dict(kind="slab", M=500, width=0.05, dt=2e-3, p=10),           # too high an order: pair by pair
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_bins_equal_stored_weights(wfp, case):
    kw = {k: case[k] for k in ("p", "W", "n_gl_local") if k in case}
    out = {}
    for mode in (2, 3):
        plan = wfp.Plan(_problem(case), case["dt"], local_mode=mode, **kw)
        assert plan.info["local_mode"] == mode and plan.info["n_pairs"] >= 112 * case["M"]
        plan.set_state(50, **_histories(plan))
        out[mode] = [plan.local_part().cpu().numpy() for _ in range(2)]
        plan.close()
    a, b = out[2][0], out[3][0]
    err = np.max(np.abs(a - b)) / np.max(np.abs(b))
    print(f"{case}: {err:.2e}", flush=True)
    assert err < TOL
    assert np.array_equal(out[2][0], out[2][1])


@pytest.mark.parametrize("case", [dict(kind="slab", M=130, width=0.02, dt=1e-3),
                                  dict(kind="slab", M=391, width=0.1, dt=2e-3, p=6),
                                  dict(kind="seam", M=300, width=0.05, dt=4e-3),
                                  dict(kind="slab", M=300, width=0.05, dt=2e-3, W=37)],
                         ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
def test_bins_gradient_equals_stored_weights(wfp, case):
    """Both gradients (the derivative sums take blocks of 16 sources and two
    histories), against the weights and derivatives stored per ordered pair."""
    import torch
    kw = {k: case[k] for k in ("p", "W") if k in case}
    prob = _problem(case)
    prob["packets"] = np.array([[1.0, 0.0, 1.0, 20.0, 0.3]])
    n = 45
    e = torch.randn(n, 3, generator=torch.Generator().manual_seed(5), dtype=torch.float64).cuda()
    got = {}
    for mode in (1, 2):
        plan = wfp.Plan(prob, case["dt"], local_mode=mode, checkpoint_every=-20, **kw)
        plan.march(n)
        got[mode] = [v.cpu().numpy() for v in plan.gradient(e)]
        plan.close()
    for a, b in zip(got[2], got[1]):
        err = np.max(np.abs(a - b)) / np.max(np.abs(b))
        print(f"{case}: {err:.2e}", flush=True)
        # 45 levels of the sums above, forward and back
        assert err < 45 * TOL


def test_bins_in_a_batch(wfp):
    """Instances by distance bins, chosen and by default, beside stored ones:
    each equals its own plan with stored weights."""
    cases = [dict(kind="slab", M=450, width=0.02, dt=1e-3), dict(kind="slab", M=129, width=0.02, dt=2e-3),
             dict(kind="slab", M=70, width=1.0, dt=2e-3)]
    modes = [0, 2, 1]
    import torch
    probs = []
    for c in cases:
        p = _problem(c)
        p["packets"] = np.array([[1.0, 0.0, 1.0, 20.0, 0.3]])
        p["x_recv"] = np.zeros(0)
        probs.append(p)
    b = wfp.Batch(probs, [c["dt"] for c in cases], per_instance=[{"local_mode": m} for m in modes])
    assert [b.plan(i).info["local_mode"] for i in range(3)] == [2, 2, 1]
    n = 30
    out = [torch.empty(s, dtype=torch.float64, device="cuda") for s in b.sizes]
    b.run(n, out)
    for i, c in enumerate(cases):
        plan = wfp.Plan(probs[i], c["dt"], local_mode=1)
        ref = plan.march(n)[0][-1].cpu().numpy()
        plan.close()
        err = np.max(np.abs(out[i].cpu().numpy() - ref)) / np.max(np.abs(ref))
        print(f"{c}: {err:.2e}", flush=True)
        assert err < n * TOL
    b.close()
