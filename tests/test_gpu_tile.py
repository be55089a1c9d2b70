"""The whole-tile step variants (lbm_step_variant_info M = 0, G = 18) at the
sizes where their tiles begin and end, against the (4, 1, 2, 1, 0, 1) variant,
which the oracle tests cover: the same expressions in the same order, so the
populations are equal bit for bit; the energy logs add the same terms in
another order (n terms: relative difference below n 2^-53)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1010_4124_amd import inputs, lbm

pytestmark = pytest.mark.gpu
P, F, R, O = 0, 1, 2, 3
SIDES = [(1.1, 0.05, 0.0, 0.9), (0.8, -0.05, 0.02, 1.05), (1.0, 0.0, 0.05, 1.0),
         (0.9, 0.1, -0.05, 0.85)]
BCS = [(P, P, P, P), (P, P, R, R), (F, F, P, P), (R, F, F, R), (O, O, P, P), (R, O, O, F)]
# widths around one, two and three tiles and their halos, heights around the rows of a tile
SHAPES = [(3, 3), (61, 4), (63, 5), (64, 7), (65, 8), (66, 9), (67, 11), (70, 17), (128, 12),
          (130, 15), (191, 13), (196, 22)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


def _variants():
    info = [lbm.lbm_step_variant_info(v) for v in range(lbm.lbm_step_variant_count())]
    tile = [v for v, i in enumerate(info) if i[5] == 0 and i[1] == 18]
    assert len(tile) >= 3 and {info[v][0] for v in tile} == {1, 2, 4}
    return tile, info.index((4, 1, 2, 1, 0, 1))


@pytest.mark.parametrize("bc", BCS)
def test_equal_to_the_carried_sum_variant_at_tile_edges(bc):
    tile, ref = _variants()
    for nx, ny in SHAPES:
        ctx = lbm.Context(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bc, side_state=SIDES)
        f = torch.from_numpy(inputs.random_f(nx, ny, seed=nx + ny)).cuda()
        ctx.variant = ref
        want, ke0 = ctx.step(f, 3, ke_log=True)
        for v in tile:
            ctx.variant = v
            got, ke = ctx.step(f, 3, ke_log=True)
            assert torch.equal(got, want), (nx, ny, lbm.lbm_step_variant_info(v))
            assert float(((ke - ke0) / ke0).abs().max()) < nx * ny * 2.0 ** -53


def test_default_variant_and_batches_of_it():
    """Small grids and batches of them get a whole-tile variant by default, and
    a batch (whatever its slots) gives what each grid alone gives."""
    tile, _ = _variants()
    bcs = [(P, P, R, R), (O, O, P, P), (F, R, P, P)]
    setups = []
    for q, (nx, ny) in enumerate(((67, 33), (130, 9), (64, 64))):
        r = inputs.random_fields(nx, ny, q)
        setups.append(inputs.Setup(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bcs[q], *r, SIDES))
    b = lbm.Batch.from_setups(setups)
    assert b.variant in tile
    f0 = b.init(*[b.pack_scalars([s.fields()[q] for s in setups]) for q in range(4)])
    for v in tile:
        b.variant = v
        for slots, chunk in ((0, 0), (3, 2)):
            b.schedule = (slots, chunk)
            out = b.step(f0, 5)
            for i, s in enumerate(setups):
                c = lbm.Context.from_setup(s)
                assert c.variant in tile
                c.variant = v
                assert torch.equal(b.view(out, i), c.step(b.view(f0, i).contiguous(), 5)), (v, i)


@pytest.mark.parametrize("shape", [(2051, 1023), (1023, 2049)])
def test_step_sums_of_a_whole_tile_variant(shape):
    """On both sides of 2^21 cells, from which on step_sums takes another
    kernel: the state of step, and the sums of that state, bit for bit."""
    tile, _ = _variants()
    nx, ny = shape
    ctx = lbm.Context(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, (P, P, R, O))
    assert ctx.variant in tile and ctx.carries_sums() == (nx * ny >= 1 << 21)
    f = torch.as_tensor(inputs.random_f(nx, ny, seed=5), device="cuda")
    want = ctx.step(f)
    for m in (None, ctx.sums(f)):
        got, sums = ctx.step_sums(f, m)
        assert torch.equal(got, want)
        assert torch.equal(sums, ctx.sums(want))


def test_very_wide_grid():
    """Past 2^24 cells per row, where every tile takes the boundary path."""
    tile, ref = _variants()
    nx = (1 << 24) + 5
    ctx = lbm.Context(nx, 1, 2e-2, 2e-2, 4e-4, 6e-4, (P, P, P, P))
    x = torch.arange(nx, dtype=torch.float64, device="cuda")[None, :] * (2e-3)
    one = torch.ones_like(x)
    f = ctx.init(one + 0.1 * torch.sin(x), 0.1 * torch.cos(x), 0 * x, one)
    ctx.variant = ref
    want = ctx.step(f)
    out = ctx.empty_f()
    for v in tile:
        ctx.variant = v
        ctx.step(f, out=out)
        assert torch.equal(out, want), v


@pytest.mark.parametrize("shape", [(201, 203), (301, 305)])
@pytest.mark.parametrize("scheme", [lbm.UPWIND1, lbm.UPWIND2])
def test_upwind_schemes_on_grids_of_higher_tiles(shape, scheme):
    """Grids whose upwind step takes tiles of 2 and of 4 rows, against the
    oracle (normwise 1e-12, the bar of the schemes' other cases)."""
    nx, ny = shape
    bc = (R, O, P, P)
    f = inputs.random_f(nx, ny, seed=9)
    p = oracle.OracleParams.make(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bc, side_state=SIDES,
                                 scheme=scheme)
    want = oracle.step(p, f, 3, nthreads=8)
    ctx = lbm.Context(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bc, side_state=SIDES, scheme=scheme)
    got, ke = ctx.step(torch.from_numpy(f).cuda(), 3, ke_log=True)
    assert np.abs(got.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    e = oracle.kinetic_y(p, f)
    assert ke[0].cpu().numpy() == pytest.approx(np.asarray(e), rel=1e-12)
