"""Whole solves at the sizes where the integration kernel changes form (GPU)."""
import numpy as np
import pytest

import synth
from oracle import bdf, chem
from tests.gpu_util import device, rel_err_above, solve_cells

pytestmark = pytest.mark.gpu


def first_species(full, n):
    """The reactions of a network among n of its species: the elements' own, then
    by first appearance in a reaction."""
    order = [full.index(a) for a in ("e-", "H", "He", "C", "N", "O", "S")]
    sides = np.concatenate([full.reactants, full.products], axis=1)
    order += [int(i) for i in dict.fromkeys(sides.ravel().tolist()) if i >= 0 and i not in order]
    keep = sorted(order[:n])
    new = np.full(full.n_species + 1, -1, np.int32)   # the last entry: no species
    new[keep] = np.arange(n)
    inside = ((sides < 0) | (new[sides] >= 0)).all(axis=1)
    return synth.Network(f"{full.name}-{n}", [full.species[i] for i in keep], full.comp[keep], full.charge[keep],
                         full.rtype[inside], new[full.reactants[inside]], new[full.products[inside]],
                         full.alpha[inside], full.beta[inside], full.gamma[inside], full.albedo)


# one wave a cell with 1, 2 or 4 tiles of 16 to a side up to 64 species, eight waves
# from 65 on
@pytest.mark.parametrize("n", [16, 17, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("precision", ["fp64", "fp32_lu"])
def test_solve_at_kernel_edges_matches_oracle(n, precision):
    import paper_2511_10558_amd as ab
    net = first_species(synth.network_for_config("net200"), n)
    g = ab.Network.from_text(net.to_text())
    cells = synth.sample_cells(net, 3, seed=n)
    cells.t_end[:] = 1e2 * 3.15576e7
    x, status, _ = solve_cells(ab, g, cells, device(), precision=precision)
    for c in range(cells.n):
        ref = bdf.solve(chem.cell_chemistry(net, cells.cell(c)), cells.x0[c], cells.t_end[c], 1e-6, 1e-20)
        assert status[c] == 0 and ref.status == bdf.OK
        # the tolerance of whole solves at rtol 1e-6 against the oracle
        assert rel_err_above(x[c], ref.x) <= 1e-4


# at these sizes and horizons some of the 40 cells' correctors fail with FP32
# factors, plain and refined (96 species: the eight-wave kernel)
@pytest.mark.parametrize("n,years", [(16, 1e3), (17, 1e3), (33, 1e6), (64, 1e6), (96, 1e6)])
def test_fp32_cells_fall_back_to_fp64_factors(n, years):
    import paper_2511_10558_amd as ab
    net = first_species(synth.network_for_config("net200"), n)
    g = ab.Network.from_text(net.to_text())
    cells = synth.sample_cells(net, 40, seed=77, t_end_yr=years)
    x, status, stats = solve_cells(ab, g, cells, device(), precision="fp32_lu", lu_reuse=0.3)
    assert (status == 0).all()
    fell = np.nonzero(stats["n_lu_fp64"])[0]
    assert len(fell) > 0 and (stats["n_lu_fp64"] <= stats["n_lu"]).all()
    for c in fell[:2]:
        ref = bdf.solve(chem.cell_chemistry(net, cells.cell(c)), cells.x0[c], cells.t_end[c], 1e-6, 1e-20)
        assert ref.status == bdf.OK and rel_err_above(x[c], ref.x) <= 1e-4


# cells interrupted (fewer slots than cells: a launch ends when a workgroup runs
# idle) and resumed, those on FP64 factors among them
@pytest.mark.parametrize("n,years", [(16, 1e3), (31, 1e4), (64, 1e4), (65, 1e4)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_lu"])
@pytest.mark.parametrize("method", ["bdf", "esdirk5"])
def test_interrupted_cells_give_the_same_bits(n, years, precision, method):
    import paper_2511_10558_amd as ab
    net = first_species(synth.network_for_config("net200"), n)
    g = ab.Network.from_text(net.to_text())
    cells = synth.sample_cells(net, 40, seed=77, t_end_yr=years)
    kw = dict(precision=precision, method=method, max_steps=3000)
    x, status, stats = solve_cells(ab, g, cells, device(), **kw)
    budget = 9 * (8 * (net.n_species * net.n_species * 6 + net.n_reactions) + 80000)   # 10 to 30 slots
    xf, sf, stf = solve_cells(ab, g, cells, device(), hbm_budget_bytes=budget, **kw)
    assert np.array_equal(sf, status) and np.array_equal(xf, x)
    assert np.array_equal(stf, stats)


def with_reactions(net, n):
    """net with its reactions repeated to n, every rate shared among its copies."""
    i = np.arange(n) % len(net.alpha)
    return synth.Network(f"{net.name}-{n}rx", net.species, net.comp, net.charge, net.rtype[i], net.reactants[i],
                         net.products[i], net.alpha[i] / np.bincount(i)[i], net.beta[i], net.gamma[i], net.albedo)


# 64 species: the one-wave kernel's dynamic LDS passes 160 KiB less its 624 bytes
# of static LDS between 562 and 564 reactions, and 160 KiB between 584 and 586
@pytest.mark.parametrize("n", [562, 564, 575, 584, 586])
@pytest.mark.parametrize("precision", ["fp64", "fp32_lu"])
def test_solve_where_the_tables_fill_the_lds(n, precision):
    import paper_2511_10558_amd as ab
    base = first_species(synth.network_for_config("net200"), 64)
    net = with_reactions(base, n)
    cells = synth.sample_cells(net, 2, seed=n, t_end_yr=1e2)
    x, status, _ = solve_cells(ab, ab.Network.from_text(net.to_text()), cells, device(), precision=precision)
    ref, _, _ = solve_cells(ab, ab.Network.from_text(base.to_text()), cells, device(), precision=precision)
    assert (status == 0).all()
    # the same chemistry, summed in another order: both within the solver's error at rtol 1e-6
    assert max(rel_err_above(x[c], ref[c]) for c in range(2)) <= 1e-4


# the largest network of 500 species that admission's LDS holds, (4 S + R) doubles
# and 232 bytes, and the smallest that is refused
@pytest.mark.parametrize("n,fits", [(18451, True), (18452, False)])
def test_largest_network(n, fits):
    import paper_2511_10558_amd as ab
    net = with_reactions(synth.network_for_config("net500"), n)
    cells = synth.sample_cells(net, 2, seed=n, t_end_yr=1e0)
    g = ab.Network.from_text(net.to_text())
    if not fits:
        with pytest.raises(ab.AbdfError, match="E_ARG.*too large"):
            solve_cells(ab, g, cells, device())
        return
    _, status, _ = solve_cells(ab, g, cells, device())
    assert (status == 0).all()


# a budget for one slot with the factors' rows unpadded (120 species: 128 doubles a
# row; padded rows would take another 16 kB)
@pytest.mark.parametrize("noalloc", [False, True])
def test_budget_of_one_unpadded_slot(noalloc):
    import paper_2511_10558_amd as ab
    net = first_species(synth.network_for_config("net200"), 120)
    S, R = net.n_species, net.n_reactions
    absJ = abs(chem.stoichiometry(net)) @ abs(chem.rate_derivative(net, np.ones(R), np.ones(S)))
    budget = 8 * (128 * 128 + 2 * 2 * 64 * 64 + R + 13 * S + absJ.nnz) + 4 * 128 + 8000
    g = ab.Network.from_text(net.to_text())
    cells = synth.sample_cells(net, 3, seed=8, t_end_yr=1e3)
    x, status, _ = solve_cells(ab, g, cells, device())
    xb, sb, _ = solve_cells(ab, g, cells, device(), hbm_budget_bytes=budget, noalloc=noalloc)
    assert (status == 0).all() and np.array_equal(sb, status) and np.array_equal(xb, x)
