"""jorge_step_noalloc (the entry point that allocates nothing) against jorge_step.

Each call takes one layer's step with the caller's state and the library's
static device scratch; a context created for the same layer with the same
options runs the same kernels over the same launch tables, so the two must
agree bitwise. Consecutive calls get smaller layers, so a call that read what
the previous one left in the scratch would show.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2310_12298_amd.jorge import Jorge, JorgeError  # noqa: E402
from paper_2310_12298_amd.workloads import gradient, initial_params  # noqa: E402

pytestmark = pytest.mark.gpu
HP = dict(lr=0.1, beta2=0.9, beta1=0.9, weight_decay=5e-5)
KINDS = ("L", "R", "mom", "mom_sgd")


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def to_dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def _compare_steps(shape, steps, **opts):
    """`steps` steps of one layer through a context and through jorge_step_noalloc; bitwise."""
    m, n = shape
    ctx = Jorge([shape], **opts)
    p_ctx = to_dev(initial_params(0, 0, shape))
    p_na = p_ctx.clone()
    a0 = 1e-6 ** -0.25
    st = {"L": torch.eye(m, device="cuda") * a0, "R": torch.eye(n, device="cuda") * a0,
          "mom": torch.zeros(shape, device="cuda"), "mom_sgd": torch.zeros(shape, device="cuda")}
    for t in range(1, steps + 1):
        g = to_dev(gradient(0, 0, t, shape, 1e-2))
        ctx.step([p_ctx], [g], **HP)
        Jorge.step_noalloc(t, p_na, g, st["L"], st["R"], st["mom"], st["mom_sgd"], **HP, **opts)
    torch.cuda.synchronize()
    assert torch.equal(p_ctx, p_na), shape
    for k in KINDS:
        assert torch.equal(ctx.get_state(0, k), st[k]), (shape, k)


def test_noalloc_matches_the_context_step_on_shrinking_layers():
    # Levels with split tiles, wave-split levels, then the small-context kernels.
    split = lambda shape: any(v[1] for v in Jorge.plan_stages([shape]).values())  # noqa: E731
    units = lambda shape: any(v[0] for v in Jorge.plan_stages([shape]).values())  # noqa: E731
    assert split((512, 1024)) and not split((256, 1152)) and not units((64, 100))
    # (256, 1152): a unit per 32 x 32 block of L G
    assert Jorge.plan_stages([(256, 1152)])["uprecond_L"][0] == (256 // 32) * (1152 // 32)
    for shape in [(512, 1024), (256, 1152), (200, 300), (64, 100), (48, 40)]:
        say("noalloc vs context", shape)
        _compare_steps(shape, 3)


def test_noalloc_options_and_interval():
    say("noalloc, interval 2, cubic term, no split")
    _compare_steps((130, 260), 3, precond_interval=2, series_order=3, split_k=False)


def test_noalloc_rejects_what_does_not_fit():
    # A 1024 x 1024 layer's workspace with split tiles is above the scratch; without split-K it fits.
    assert Jorge.plan([(1024, 1024)]) > 64 << 20 > Jorge.plan([(1024, 1024)], split_k=False)
    x = torch.zeros((1024, 1024), device="cuda")
    L = torch.eye(1024, device="cuda")
    before = L.clone()
    with pytest.raises(JorgeError) as e:
        Jorge.step_noalloc(1, x, x, L, L.clone(), x.clone(), x.clone(), **HP)
    assert e.value.status == -4
    assert torch.equal(L, before)
    with pytest.raises(JorgeError) as e:
        Jorge.step_noalloc(0, x, x, L, L.clone(), x.clone(), x.clone(), **HP)
    assert e.value.status == -1
