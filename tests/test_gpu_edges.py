"""Sizes at which the list build, its species grouping and the totals change
the way they are computed (edges of workgroups, of the one-workgroup scan, of
the cell capacity of a wave and of its sharing over several waves).

* The list and the per-species grouping behind the network: energies, forces
  and virial against the FP64 oracle to the FP32 bars of tests/parity.py.
* The total energy against the exact sum of the returned atomic energies: the
  library sums FP32 values in FP64 with compensation, so only the final
  rounding remains (relative 2^-52; 1e-14 allows for cancellation to a
  hundredth of the summed magnitude).
"""
import math

import numpy as np
import pytest

import parity
from paper_2310_08439_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2310_08439_amd import tmd
    c = tmd.Context(0)
    yield c
    c.close()


def _evaluate(ctx, spec, s):
    import torch
    from paper_2310_08439_amd import tmd
    pos = torch.tensor(s.pos, dtype=torch.float64, device="cuda")
    sp = torch.tensor(s.species, dtype=torch.int32, device="cuda")
    ev = tmd.Evaluator(spec, s.n, s.box, precision=tmd.FP32, ctx=ctx)
    E, Ea, F, W = ev.energy_forces(pos, sp, s.box)
    again = ev.energy_forces(pos, sp, s.box)  # the launch counters start at zero again
    assert again[0] == E and np.array_equal(again[3], W)
    return E, Ea.cpu().numpy().astype(np.float64), F.cpu().numpy().astype(np.float64), W


def _check(ctx, spec, s):
    print(f"[case] {s.n} atoms, box {s.box}, {spec.n_species} species", flush=True)
    E, Ea, F, W = _evaluate(ctx, spec, s)
    assert abs(E - math.fsum(Ea)) <= 1e-14 * float(np.abs(Ea).sum())
    parity.check_fp32(E, Ea, F, W, s, spec)


# one atom; one summing workgroup and its last size; two; several with a remainder
@pytest.mark.parametrize("n", [1, 2, 255, 257, 2047, 2048, 2049, 4097])
def test_totals_and_grouping(ctx, n):
    s = inputs.make_system("fcc", 3.61, (11, 10, 10), 0.05, 3, seed=n)
    keep = np.sort(np.random.default_rng(n).permutation(s.n)[:n])
    s = inputs.System(pos=s.pos[keep], species=s.species[keep], box=s.box, masses=s.masses)
    _check(ctx, inputs.make_model(3, 8, 3, [32], 5.0, seed=7), s)


# cell grids on both sides of the 16,384 cells that one workgroup scans:
# 25 x 25 x 26 = 16,250 and 26^3 = 17,576 cells of a dilute gas
@pytest.mark.parametrize("cells", [(25, 25, 26), (26, 26, 26)])
@pytest.mark.parametrize("n_species", [1, 3])
def test_cell_grid_of_the_scan(ctx, cells, n_species):
    rng = np.random.default_rng(cells[0] + n_species)
    spec = inputs.make_model(n_species, 8, 2, [32], 3.0, seed=8, r_min=1.0)
    box = np.array(cells) * 3.001
    n = 4500  # at least a quarter of the cells, or the grid is coarsened
    pos = rng.uniform(0.0, 1.0, size=(n, 3)) * box
    s = inputs.System(pos=pos, species=rng.integers(0, n_species, n).astype(np.int32), box=box,
                      masses=np.ones(n_species))
    # a random gas has close pairs: forces beyond the crystal's, so the bars scale with the largest force
    import oracle
    E, Ea, F, W = _evaluate(ctx, spec, s)
    Er, Ear, Fr, Wr = oracle.energy_forces(spec, s.pos, s.species, s.box)
    scale = max(1.0, float(np.abs(Fr).max()))
    assert abs(E - math.fsum(Ea)) <= 1e-14 * float(np.abs(Ea).sum())
    assert np.abs(Ea - Ear).max() <= parity.E_FP32 * scale
    assert np.abs(F - Fr).max() <= parity.FMAX_FP32 * scale


# one cell of 1 to 65 atoms (65: past what a wave tracks) shared over sixteen
# waves, and two cells per edge
@pytest.mark.parametrize("n", [1, 3, 15, 16, 17, 63, 64, 65])
@pytest.mark.parametrize("edge", [5.2, 10.4])
def test_shared_cells(ctx, n, edge):
    rng = np.random.default_rng(n)
    grid = np.stack(np.meshgrid(*[np.arange(5)] * 3, indexing="ij"), -1).reshape(-1, 3)
    pos = (grid[rng.permutation(125)[:n]] + 0.5 + rng.uniform(-0.2, 0.2, size=(n, 3))) * (edge / 5)
    s = inputs.System(pos=pos, species=(np.arange(n) % 2).astype(np.int32), box=np.full(3, edge), masses=np.ones(2))
    spec = inputs.make_model(2, 8, 3, [32], 5.0, seed=9, r_min=0.5)
    import oracle
    E, Ea, F, W = _evaluate(ctx, spec, s)
    Er, Ear, Fr, Wr = oracle.energy_forces(spec, s.pos, s.species, s.box)
    # sums over up to ~500 neighbours of terms up to 1: the bars scale with the
    # neighbour count relative to the ~50 of the configurations they were set for
    scale = max(1.0, n * 4.19 * 125.0 / edge ** 3 / 50.0) * max(1.0, float(np.abs(Fr).max()))
    assert np.abs(Ea - Ear).max() <= parity.E_FP32 * scale
    assert np.abs(F - Fr).max() <= parity.FMAX_FP32 * scale
