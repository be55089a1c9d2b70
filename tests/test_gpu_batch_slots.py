"""slots_per_xcd of the whole-tile batch variants: a grid of 8 s workgroups that
loop over the work list gives what one workgroup per tile gives, bit for bit,
and has no more than those workgroups."""
import pytest
import torch

from paper_1010_4124_amd import inputs, lbm

pytestmark = pytest.mark.gpu
P, F, R, O = 0, 1, 2, 3
SIDES = [(1.1, 0.05, 0.0, 0.9), (0.8, -0.05, 0.02, 1.05), (1.0, 0.0, 0.05, 1.0),
         (0.9, 0.1, -0.05, 0.85)]
BCS = [(P, P, R, R), (O, O, P, P), (F, R, P, P), (R, R, O, F)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


def _variants():
    info = [lbm.lbm_step_variant_info(v) for v in range(lbm.lbm_step_variant_count())]
    return [v for v, i in enumerate(info) if i[5] == 0 and i[1] == 18]


def _batch(shapes):
    setups = [inputs.Setup(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, BCS[q % 4],
                           *inputs.random_fields(nx, ny, q), SIDES)
              for q, (nx, ny) in enumerate(shapes)]
    b = lbm.Batch.from_setups(setups)
    return b, b.init(*[b.pack_scalars([s.fields()[q] for s in setups]) for q in range(4)])


@pytest.mark.parametrize("v", _variants())
def test_same_result_and_energy_log(v):
    b, f0 = _batch([(67, 33), (130, 9), (64, 64), (191, 22), (3, 3)])
    b.variant = v
    want, ke0 = b.step(f0, 5, ke_log=True)
    for slots, chunk in ((1, 0), (1, 2), (2, 4), (5, 0), (1 << 20, 0)):
        b.schedule = (slots, chunk)
        got, ke = b.step(f0, 5, ke_log=True)
        assert torch.equal(got, want) and torch.equal(ke, ke0), (slots, chunk)


def test_the_slots_limit_the_workgroups():
    """512 tiles of 4 rows: 64 rounds of 8 workgroups, or all at once."""
    b, f0 = _batch([(256, 512)])
    b.variant = next(v for v in _variants() if lbm.lbm_step_variant_info(v)[0] == 4)
    out, ms = b.empty_f(), []
    for slots in (0, 1):
        b.schedule = (slots, 0)
        b.step(f0, 10, out=out)
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        b.step(f0, 20, out=out)
        e[1].record()
        e[1].synchronize()
        ms.append(e[0].elapsed_time(e[1]))
    assert ms[1] > 4 * ms[0], ms
