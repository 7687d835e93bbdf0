"""Which of a right-hand side's state buffers holds its current state, over the
calls that can leave the host and the device with different counts of the
launches that swapped them (two steps per launch swap two buffers once)."""
import pytest
import torch

from paper_2505_03352_amd import YO_BOTH, _abi
from paper_2505_03352_amd.plan import advance_many, plan_for
from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu_available():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _abi.lib()


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("tb", [1, 2])
def test_fields_set_after_a_new_binding_are_the_ones_stepped(tb):
    """A plan bound again, without a reset, starts at step 0 of a cleared
    workspace: fields set then are what the next steps read."""
    dev = configs.micro(n_steps=40)
    p = plan_for(dev, time_blocking=tb)
    gen = torch.Generator(device="cuda").manual_seed(1)
    e, h = (torch.randn(p.shape, generator=gen, device="cuda") for _ in range(2))
    out = {}
    for before in (0, 2, 3):                 # 0, 1 and 2 launches before the new binding
        print(f"[gpu] bind again tb={tb} after {before} steps", flush=True)
        p.reset(YO_BOTH)
        p.advance(YO_BOTH, before)
        p.bind()
        p.set_background(torch.as_tensor(dev.kappa_bg, dtype=torch.float32),
                         torch.as_tensor(dev.mask_hr, dtype=torch.float32))
        p.set_fields(0, e, h)
        assert _same(p.get_fields(0), (e, h))
        p.advance(YO_BOTH, 5)
        out[before] = p.get_fields(0)
    assert out[0][0].abs().max() > 0
    for before in (2, 3):
        assert _same(out[before], out[0])
    p.close()


@pytest.mark.parametrize("tb", [1, 2])
def test_a_side_keeps_its_fields_while_the_other_runs(tb):
    """The forward run's state stays readable through an adjoint run whose
    steps go in other numbers of launches: 20 for 40 steps in one call, 23 in
    calls of 7."""
    dev = configs.micro(n_steps=41)
    p = plan_for(dev, time_blocking=tb)
    print(f"[gpu] forward state through an adjoint run tb={tb}", flush=True)
    for steps, chunk in ((41, 40), (40, 7), (41, 41)):
        p.reset(1)
        advance_many([p], [1], steps, chunk=chunk, use_graph=False)
        fwd = p.get_fields(0)
        assert fwd[0].abs().max() > 0
        p.reset(2)
        assert _same(p.get_fields(0), fwd)
        for n in (2, 1, 37):
            advance_many([p], [2], n, chunk=7, use_graph=False)
            assert _same(p.get_fields(0), fwd)
        adj = p.get_fields(1)
        p.reset(1)
        assert p.get_fields(0)[0].abs().max() == 0
        assert _same(p.get_fields(1), adj)
    p.close()


@pytest.mark.parametrize("tb,n", [(1, 2), (1, 3), (2, 2), (2, 5)])
def test_fields_after_a_caller_replays_captured_steps(tb, n):
    """Steps a caller captured and replays are counted on the device alone."""
    dev = configs.micro(n_steps=600)
    q = plan_for(dev, time_blocking=tb)
    q.reset(YO_BOTH)
    p = plan_for(dev, time_blocking=tb)
    p.reset(YO_BOTH)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        p.advance(YO_BOTH, n)
    p.reset(YO_BOTH)
    for k in range(4):
        print(f"[gpu] replay {k} of {n} captured steps tb={tb}", flush=True)
        g.replay()
        q.advance(YO_BOTH, n)
        torch.cuda.synchronize()
        for r in range(p.n_rhs):
            assert q.get_fields(r)[0].abs().max() > 0
            assert _same(p.get_fields(r), q.get_fields(r))
    p.close()
    q.close()
