"""jorge_step_noalloc keeps the plans of the last few kinds of layer: calls that
alternate between layers and options, come back after their plan was dropped,
follow a layer whose gradient was not finite, or come from two threads on two
streams, each equal a context's step bitwise."""
import math
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2310_12298_amd.jorge import Jorge  # noqa: E402
from paper_2310_12298_amd.workloads import gradient, initial_params  # noqa: E402

pytestmark = pytest.mark.gpu
HP = dict(lr=0.1, beta2=0.9, beta1=0.9, weight_decay=5e-5)
KINDS = ("L", "R", "mom", "mom_sgd")
SPLIT = (512, 1024)     # its levels have split tiles, so the scratch holds a split workspace


def to_dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


class Pair:
    """One layer stepped through a context and through jorge_step_noalloc."""

    def __init__(self, shape, seed=0, **opts):
        self.shape, self.opts, self.seed, self.t = shape, opts, seed, 0
        self.ctx = Jorge([shape], **opts)
        self.p_ctx = to_dev(initial_params(seed, 0, shape))
        self.p = self.p_ctx.clone()
        m, n = shape
        a0 = 1e-6 ** -0.25
        self.st = [torch.eye(m, device="cuda") * a0, torch.eye(n, device="cuda") * a0,
                   torch.zeros(shape, device="cuda"), torch.zeros(shape, device="cuda")]

    def lone(self, value=None):
        """A step of the noalloc side alone on a copy of its state (value: one bad gradient element)."""
        g = to_dev(gradient(self.seed, 9, 1, self.shape, 1e-2))
        if value is not None:
            g[0, 0] = value
        Jorge.step_noalloc(1, self.p.clone(), g, *(x.clone() for x in self.st), **HP, **self.opts)

    def step(self):
        self.t += 1
        g = to_dev(gradient(self.seed, 0, self.t, self.shape, 1e-2))
        self.ctx.step([self.p_ctx], [g], **HP)
        Jorge.step_noalloc(self.t, self.p, g, *self.st, **HP, **self.opts)

    def check(self):
        torch.cuda.synchronize()
        assert torch.equal(self.p_ctx, self.p), (self.shape, self.opts)
        for k, v in zip(KINDS, self.st):
            assert torch.equal(self.ctx.get_state(0, k), v), (self.shape, self.opts, k)


def test_alternating_layers_and_options():
    assert any(v[1] for v in Jorge.plan_stages([SPLIT]).values())
    pairs = [Pair(SPLIT), Pair((130, 260)), Pair((130, 260), symmetrize=False), Pair((130, 260), precond_interval=2),
             Pair((48, 40)), Pair((100, 70)), Pair((33, 577)), Pair((256, 300), series_order=3)]
    for _ in range(3):
        for p in pairs:
            p.step()
    for p in pairs:
        p.step()
        p.step()        # the same layer twice in a row finds its tables in the scratch
        p.check()


def test_a_dropped_plan_is_built_again():
    first = Pair((70, 90))
    first.step()
    for i in range(20):
        Pair((40 + i, 65)).step()
    first.step()
    first.check()


@pytest.mark.parametrize("shape", [(70, 301), (33, 47), (100, 65), SPLIT])
@pytest.mark.parametrize("value", [math.nan, math.inf])
def test_a_non_finite_step_leaves_nothing_behind(shape, value):
    p = Pair(shape)
    p.step()
    p.lone(value)       # the padding and the workspace now hold what it left
    p.step()
    p.check()


def test_two_threads_two_streams():
    pairs = [Pair((130, 260), seed=1), Pair((64, 100), seed=2)]
    grads = [[to_dev(gradient(p.seed, 0, t, p.shape, 1e-2)) for t in range(1, 7)] for p in pairs]
    torch.cuda.synchronize()
    errors = []

    def work(p, gs):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for t, g in enumerate(gs, 1):
                    Jorge.step_noalloc(t, p.p, g, *p.st, **HP, **p.opts)
        except Exception as e:   # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=a) for a in zip(pairs, grads)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors
    for p, gs in zip(pairs, grads):
        for g in gs:
            p.ctx.step([p.p_ctx], [g], **HP)
        p.check()
