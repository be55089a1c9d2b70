"""Grids so tall and narrow that their tiles exceed one launch (2^32
work-items): the state repeats every 40 rows, so each period equals that of a
tall grid of one launch bit for bit."""
import pytest
import torch

from paper_1010_4124_amd import lbm

pytestmark = pytest.mark.gpu
NY, TALL, PERIOD = 33_600_000, 100_000, 40
CELL = (2e-2, 2.5e-2, 4e-4, 6e-4)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


def _fields(ny):
    y = torch.arange(PERIOD, dtype=torch.float64, device="cuda")
    s, c = torch.sin(0.3 * y), torch.cos(0.2 * y)
    return [t.repeat(ny // PERIOD)[:, None].contiguous()
            for t in (1 + 0.1 * s, 0.1 * c, 0.1 * s * c, 1 + 0.05 * c)]


def _same(out, want):
    return bool((out.view(19, -1, PERIOD) == want[:, :PERIOD].reshape(19, 1, PERIOD)).all())


@pytest.mark.parametrize("scheme", [lbm.WENO5, lbm.UPWIND1])
def test_default_step_of_a_very_tall_grid(scheme):
    small = lbm.Context(1, TALL, *CELL, scheme=scheme)
    want = small.step(small.init(*_fields(TALL)), 2)
    ctx = lbm.Context(1, NY, *CELL, scheme=scheme)
    assert _same(ctx.step(ctx.init(*_fields(NY)), 2), want)


def test_default_batch_step_of_a_very_tall_grid():
    small = lbm.Context(1, TALL, *CELL)
    want = small.step(small.init(*_fields(TALL)), 2)
    b = lbm.Batch([lbm.LbmParams.make(1, NY, *CELL)])
    f = b.init(*[t.reshape(-1) for t in _fields(NY)])
    assert _same(b.step(f, 2), want)
