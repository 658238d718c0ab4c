"""Contexts of small factors only (one or two launches per step, matrices in LDS)
against the fp64 oracle, from injected states that do not commute with the
gradient's statistics.

The gates are those of one step (tests/parity_metrics.py: 1e-5 on every tensor,
1e-3 on the factors' informative part, 1e-4 on the applied step), and 2e-6 on the
state: products of depth up to 128 in fp32 are off by about 1e-7, and an update chains
eight of them.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import JorgeOracle  # noqa: E402
from paper_2310_12298_amd.jorge import Jorge  # noqa: E402
from parity_metrics import STEP, check_layer  # noqa: E402

pytestmark = pytest.mark.gpu
HP = dict(lr=0.1, beta2=0.9, beta1=0.9, weight_decay=5e-4)
# Edges of the 16- and 32-wide blocks and of both size classes, single rows and columns.
UP_TO_64 = [(1, 1), (1, 64), (64, 1), (31, 33), (32, 32), (33, 64), (64, 64), (17, 48)]
UP_TO_128 = [(65, 1), (1, 128), (97, 96), (128, 128), (127, 65), (96, 33), (32, 128), (64, 64)]
# Factors up to 64 share a workgroup: k up to and above 64 side by side, and an odd number of them.
PAIRED_128 = UP_TO_128 + [(64, 127), (90, 64), (31, 97), (128, 17), (64, 50), (65, 20), (20, 20)]


def off_by_one_float(x):
    """A contiguous device copy of x that starts one float past an aligned address."""
    buf = torch.empty(x.size + 1, dtype=torch.float32, device="cuda")
    view = buf[1:].view(*x.shape)
    view.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return view


def state(rng, m, n, sigma):
    out = []
    for d, k in ((m, n), (n, m)):
        s = rng.standard_normal((d, d))
        out.append(((np.eye(d) + 0.2 * (s + s.T) / np.sqrt(2 * d)) * (k * sigma * sigma) ** -0.25).astype(np.float32))
    return out + [rng.standard_normal((m, n)).astype(np.float32) * np.float32(1e-3 / sigma ** 0.5),
                  rng.standard_normal((m, n)).astype(np.float32) * np.float32(sigma)]


@pytest.mark.parametrize("shapes", [UP_TO_64, UP_TO_128, PAIRED_128], ids=["64", "128", "paired"])
@pytest.mark.parametrize("update", [True, False])
@pytest.mark.parametrize("symmetrize,order", [(True, 2), (True, 3), (False, 2), (False, 3)])
def test_one_step_from_an_injected_state(shapes, update, symmetrize, order):
    if shapes is not UP_TO_64 and not symmetrize:
        pytest.skip("contexts above 64 need symmetric factors to run in LDS")
    rng = np.random.default_rng([len(shapes), update, symmetrize, order, shapes[0][0]])
    sigma = 1e-2
    kw = dict(precond_interval=1 if update else 7, symmetrize=symmetrize, series_order=order)
    opt, orc = Jorge(shapes, **kw), JorgeOracle(shapes, **kw)
    opt.t = orc.t = 8
    theta, grads = [], []
    for l, (m, n) in enumerate(shapes):
        st = state(rng, m, n, sigma)
        for kind, v in zip(("L", "R", "mom", "mom_sgd"), st):
            opt.set_state(l, kind, torch.from_numpy(v))
        o = orc.layers[l]
        o.L, o.R, o.m, o.m_sgd = (v.astype(np.float64) for v in st)
        theta.append(rng.standard_normal((m, n)).astype(np.float32))
        grads.append((rng.standard_normal((m, n)) * sigma).astype(np.float32))
    pg = [off_by_one_float(x) for x in theta]
    opt.set_timing(True)
    opt.step(pg, [off_by_one_float(x) for x in grads], **HP)
    launches = {k: v[1] for k, v in opt.read_timing().items() if v[1]}
    # the whole step: one kernel up to 64; else one for the factors and one for the rest
    assert launches == {"lds_chain": 1 if shapes is UP_TO_64 or not update else 2}
    prev = [x.astype(np.float64) for x in theta]
    po = orc.step(prev, grads, HP["lr"], HP["beta2"], HP["beta1"], HP["weight_decay"])
    for l in range(len(shapes)):
        o = orc.layers[l]
        got = {k: opt.get_state(l, k).cpu().numpy() for k in ("L", "R", "mom", "mom_sgd")}
        check_layer(got, {"L": o.L, "R": o.R, "mom": o.m, "mom_sgd": o.m_sgd}, pg[l].cpu().numpy(), po[l], prev[l],
                    HP["lr"], HP["weight_decay"], STEP, f"layer {l} {shapes[l]}")
        for k, want in (("L", o.L), ("R", o.R), ("mom", o.m), ("mom_sgd", o.m_sgd)):
            err = np.linalg.norm(got[k] - want) / np.linalg.norm(want)
            assert err <= 2e-6, (l, shapes[l], k, err)
        if symmetrize:
            assert np.array_equal(got["L"], got["L"].T) and np.array_equal(got["R"], got["R"].T), l


def test_paired_sizes():
    small = [(k, d) for m, n in PAIRED_128 for d, k in ((m, n), (n, m)) if d <= 64]
    assert len(small) % 2 and any(k > 64 for k, _ in small) and any(k <= 64 for k, _ in small)


@pytest.mark.parametrize("layers", [1, 2, 7])
def test_a_factor_does_not_depend_on_its_neighbour(layers):
    """A layer's factors up to 64 give the same bits beside deep and shallow factors, alone and in pairs."""
    rng = np.random.default_rng(9)
    shape = (48, 40)
    st, g = state(rng, *shape, 1e-2), (rng.standard_normal(shape) * 1e-2).astype(np.float32)
    out = []
    for shapes in ([(96, 96), shape], [shape] * layers + [(128, 40)], [(60, 120)] * layers + [shape, (70, 9)]):
        opt, l = Jorge(shapes), shapes.index(shape)
        for kind, v in zip(("L", "R", "mom", "mom_sgd"), st):
            opt.set_state(l, kind, torch.from_numpy(v))
        params = [torch.zeros(s, device="cuda") for s in shapes]
        grads = [torch.ones(s, device="cuda") for s in shapes]
        grads[l] = torch.from_numpy(g).cuda()
        opt.step(params, grads, **HP)
        out.append([opt.get_state(l, k) for k in ("L", "R", "mom")] + [params[l]])
    for other in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], other))


def test_layers_of_several_batches_step_alike():
    """Layers past the first 256 (a launch's worth of pointers) get their own tensors."""
    shapes = [(40, 96)] * 300
    rng = np.random.default_rng(5)
    theta, g = rng.standard_normal((40, 96)).astype(np.float32), rng.standard_normal((40, 96)).astype(np.float32)
    opt = Jorge(shapes)
    params = [torch.from_numpy(theta).cuda() for _ in shapes]
    grads = [torch.from_numpy(g * np.float32(1 + i % 3)).cuda() for i in range(300)]
    for _ in range(2):
        opt.step(params, grads, **HP)
    for i in range(3, 300):
        assert torch.equal(params[i], params[i % 3]), i
    assert not torch.equal(params[0], params[1])


def test_stage_flops_keep_updates_and_preconditioning_apart():
    m, n = 40, 96
    fl = Jorge([(m, n)] * 3).stage_flops()
    for stage in ("precond", "uprecond"):       # on steps between updates, and on updating ones
        assert fl[stage + "_L"] == 3 * 2 * m * m * n and fl[stage + "_R"] == 3 * 2 * m * n * n
    # Algorithm 2's products, symmetric ones once: H H^T, A^2, A^4, then X, X X and A P
    factor = lambda d, k: d * d * k + 2 * d ** 3 + 6 * d ** 3  # noqa: E731
    assert fl["lds_chain"] == 3 * (factor(m, n) + factor(n, m))
