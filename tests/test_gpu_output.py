"""GPU parity of the output stage (Methods, end of "Accelerated Docking with
QuickVina 2-GPU 2.1"; last steps of Supplementary Algorithm 2) against the
oracle: exact selection and order on constructed chain sets without
refinement (one and two atoms per lane, several jobs), refined modes on a
smooth objective, and validity of the modes of a real dock."""
import numpy as np
import pytest

from gpu_util import cpu_dof, e_tol
from paper_2506_20043_amd import synth as S
from test_oracle_output import cluster_set, _rmsd

pytestmark = pytest.mark.gpu
KAPPA = 10.0


@pytest.fixture(scope="module")
def pv_ctx():
    import paper_2506_20043_amd as pv
    return pv.Context(0)


def _setup(oracle, pv_ctx, rx, rt, box, mols):
    import paper_2506_20043_amd as pv
    grids = pv.build_grids(pv_ctx, rx, rt, [box], penalty_slope=KAPPA)
    ligs = pv.Ligands(pv_ctx, mols)
    dims, org = grids.info(0)
    G = oracle.Grid.build(rx, rt, box.center.astype(np.float64), box.size.astype(np.float64), box.spacing,
                          kappa=KAPPA)
    return grids, ligs, G


def _run(pv, pv_ctx, grids, ligs, jobs, chains, dof, e, **kw):
    plan = pv.Plan(pv_ctx, grids, ligs, jobs, pv.dock_params(chains=chains, steps=0))
    stride = ligs.dof_stride
    d = np.zeros((len(jobs) * chains, stride), np.float32)
    d[:, :dof.shape[-1]] = dof.reshape(-1, dof.shape[-1])
    out = pv.output_stage(plan, np.float32(e).reshape(-1), d, pv.output_params(**kw))
    res = {k: v.cpu().numpy() for k, v in out.items()}
    plan.close()
    return res


def _compare(oracle, L, G, res, dof, e, j, chains, modes, refine, cut=1.0):
    ref = oracle.output_stage(L, G, dof[j], e[j], modes=modes, refine_max_iter=refine, rmsd_cut=cut)
    n = len(ref["chain"])
    assert ref["rmsd_margin"] > 1e-3 and ref["energy_gap"] > 1e-3, "constructed set has a near tie"
    assert res["n_modes"][j] == n
    assert list(res["mode_chain"][j, :n]) == list(ref["chain"])
    assert np.all(res["mode_chain"][j, n:] == -1) and np.all(np.isnan(res["mode_e"][j, n:]))
    assert np.all(np.abs(res["mode_e"][j, :n] - ref["e"]) <= e_tol(ref["e"]))
    assert np.all(np.abs(res["mode_affinity"][j, :n] - ref["affinity"]) <= e_tol(ref["affinity"]))
    nd = L.ndof
    assert np.abs(res["mode_dof"][j, :n, :nd] - ref["dof"]).max() <= 1e-5
    assert np.all(res["mode_dof"][j, :, nd:] == 0.0)


def test_output_matches_oracle_without_refinement(oracle, pv_ctx):
    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    mols = S.make_ligands(cfg)
    grids, ligs, G = _setup(oracle, pv_ctx, rx, rt, bxs[0], mols)
    L = oracle.Ligand(mols[0].xyz, mols[0].types, mols[0].bonds, mols[0].rotatable)
    g = np.random.default_rng(71)
    sizes = [[2, 1, 4, 3, 1, 2, 5, 1, 3, 2, 2, 4], [2] * 12, [12, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 2]]
    dof, e = [], []
    for sz in sizes:
        d, _, ee = cluster_set(L, G, g, 12, sz)
        order = np.argsort(g.random(len(d)))[:24]          # 24 chains per job
        dof.append(d[order]); e.append(ee[order])
    dof, e = np.stack(dof), np.stack(e)
    for modes in (8, 20):
        res = _run(pv, pv_ctx, grids, ligs, [(0, 0)] * 3, 24, dof, e, modes=modes, refine_max_iter=0)
        for j in range(3):
            _compare(oracle, L, G, res, dof, e, j, 24, modes, 0)


def test_output_two_atoms_per_lane(oracle, pv_ctx):
    """A 70-atom ligand runs the two-atoms-per-lane kernel."""
    import paper_2506_20043_amd as pv
    g = np.random.default_rng(72)
    rx, rt = S.receptor(g, 2500, 40.0)
    box = S.Box(np.full(3, 20.0, np.float32), np.full(3, 26.0, np.float32), 0.375)
    mol = S.tree_ligand(g, 70, 9)
    grids, ligs, G = _setup(oracle, pv_ctx, rx, rt, box, [mol])
    L = oracle.Ligand(mol.xyz, mol.types, mol.bonds, mol.rotatable)
    dof, _, e = cluster_set(L, G, g, 9, [2, 3, 1, 2, 1, 4, 2, 1, 2])
    res = _run(pv, pv_ctx, grids, ligs, [(0, 0)], len(e), dof[None], e[None], modes=6, refine_max_iter=0)
    _compare(oracle, L, G, res, dof[None], e[None], 0, len(e), 6, 0)


def test_output_refined_on_smooth_objective(oracle, pv_ctx):
    """No receptor, C_P atoms, at most 5 bonds across: the intra energy is
    smooth, so FP32 and FP64 BFGS refine to the same minima; the intra-only
    objective leaves t and q alone, so the clusters stay apart."""
    import paper_2506_20043_amd as pv
    from test_oracle_search import _diameter
    g = np.random.default_rng(73)
    while True:
        m = S.tree_ligand(g, 9, 4)
        if m.n_tors >= 3 and _diameter(9, m.bonds) <= 5:
            break
    mol = S.Molecule(m.xyz, np.full(9, 1, np.int32), m.bonds, m.rotatable, m.n_tors)
    box = S.Box(np.zeros(3, np.float32), np.full(3, 40.0, np.float32), 1.0)
    grids, ligs, _ = _setup(oracle, pv_ctx, np.zeros((0, 3), np.float32), np.zeros(0, np.uint8), box, [mol])
    dims, org = grids.info(0)
    G = oracle.Grid(np.zeros((8, dims[2], dims[1], dims[0])), dims, org, 1.0, kappa=KAPPA)
    L = oracle.Ligand(mol.xyz, mol.types, mol.bonds, mol.rotatable)
    dof, _, e = cluster_set(L, G, g, 6, [3, 2, 1, 4, 2, 3], sep=4.0, spread=0.01, margin=9.0)
    res = _run(pv, pv_ctx, grids, ligs, [(0, 0)], len(e), dof[None], e[None], modes=6, refine_max_iter=300)
    ref = oracle.output_stage(L, G, dof, e, modes=6, refine_max_iter=300, rmsd_cut=1.0,
                              bfgs=oracle.bfgs_params(max_iter=300))
    n = len(ref["chain"])
    assert res["n_modes"][0] == n == 6
    # refined energies of different clusters may coincide, so compare each
    # selected chain's refined energy, and each side's order
    got = dict(zip(res["mode_chain"][0, :n], res["mode_e"][0, :n]))
    want = dict(zip(ref["chain"], ref["e"]))
    assert set(got) == set(want)
    for c in want:
        assert abs(got[c] - want[c]) <= 1e-3, (c, got[c], want[c])
    assert np.all(np.diff(res["mode_e"][0, :n]) >= 0)


def test_output_of_a_dock_is_valid(oracle, pv_ctx):
    """Modes of a real dock (tiny configuration): sorted, separated by the
    cut, each re-scored by the oracle to its energy and affinity, never
    above its source chain's energy, unit quaternions."""
    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    mols = S.make_ligands(cfg)
    grids, ligs, G = _setup(oracle, pv_ctx, rx, rt, bxs[0], mols)
    L = oracle.Ligand(mols[0].xyz, mols[0].types, mols[0].bonds, mols[0].rotatable)
    plan = pv.Plan(pv_ctx, grids, ligs, [(0, 0), (0, 0)], pv.dock_params(chains=64, steps=60, seed=S.philox_seed(cfg)))
    out = plan.run()
    modes = pv.output_stage(plan, out["chain_best_e"], out["chain_best_dof"])
    res = {k: v.cpu().numpy() for k, v in modes.items()}
    cbe = out["chain_best_e"].cpu().numpy().reshape(2, 64)
    plan.close()
    for j in range(2):
        n = int(res["n_modes"][j])
        assert 1 <= n <= 20
        e = res["mode_e"][j, :n]
        assert np.all(np.diff(e) >= 0)
        ch = res["mode_chain"][j, :n]
        assert len(set(ch)) == n and np.all((ch >= 0) & (ch < 64))
        xs = []
        for o in range(n):
            d = cpu_dof(res["mode_dof"][j, o, :L.ndof])
            assert np.linalg.norm(d[3:7]) == pytest.approx(1.0, abs=1e-5)
            r = L.score_grad(G, d)
            slack = 0.01 if r["min_cut"] < 1e-4 else 0.0
            assert abs(e[o] - r["e"]) <= e_tol(r["e"]) + slack
            aff = r["e_inter"] / (1 + 0.0585 * L.n_tors)
            assert abs(res["mode_affinity"][j, o] - aff) <= e_tol(aff) + slack
            assert e[o] <= cbe[j, ch[o]] + e_tol(cbe[j, ch[o]])
            xs.append(r["xyz"])
        for o in range(n):
            for p in range(o):
                assert _rmsd(xs[o], xs[p]) >= 1.0 - 1e-3


@pytest.mark.parametrize("n_atoms, chains, modes", [(20, 1, 1), (20, 7, 3), (20, 9, 20), (20, 65, 32), (70, 33, 20)])
def test_output_independent_of_the_waves(oracle, pv_ctx, n_atoms, chains, modes):
    """A few jobs run eight waves each, more jobs than CUs four: batches of the clustering, refinements and filter
    rows fall on other waves, and every job's modes stay the same bit for bit."""
    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    mols = [S.tree_ligand(np.random.default_rng(5), n_atoms, 6)]
    grids, ligs, G = _setup(oracle, pv_ctx, rx, rt, bxs[0], mols)
    params = pv.dock_params(chains=chains, steps=8, seed=3)
    dock = pv.dock(pv_ctx, grids, ligs, [(0, 0)], params)
    # pairs of near copies among the chains, so that the clustering drops some
    dof, e = dock["chain_best_dof"].cpu().numpy(), dock["chain_best_e"].cpu().numpy()
    dof[1::3, :] = dof[:-1:3, :][:len(dof[1::3])]
    dof[1::3, 0] += np.float32(0.2)
    runs = []
    for n in (2, 300):
        res = _run(pv, pv_ctx, grids, ligs, [(0, 0)] * n, chains, np.stack([dof] * n), np.stack([e] * n), modes=modes)
        for k, v in res.items():
            assert np.array_equal(v, np.stack([v[0]] * n), equal_nan=v.dtype.kind == "f"), k
        runs.append(res)
    for k in runs[0]:
        assert np.array_equal(runs[0][k][0], runs[1][k][0], equal_nan=runs[0][k].dtype.kind == "f"), k
    assert 1 <= runs[0]["n_modes"][0] <= modes


def test_output_rejects(pv_ctx):
    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    grids = pv.build_grids(pv_ctx, rx, rt, bxs, penalty_slope=KAPPA)
    ligs = pv.Ligands(pv_ctx, S.make_ligands(cfg))
    plan = pv.Plan(pv_ctx, grids, ligs, [(0, 0)], pv.dock_params(chains=8, steps=0))
    e = np.zeros(8, np.float32)
    d = np.zeros((8, ligs.dof_stride), np.float32)
    d[:, 3] = 1.0
    for kw in ({"modes": 0}, {"modes": 33}, {"rmsd_cut": -1.0}, {"rmsd_cut": float("nan")},
               {"refine_max_iter": -1}, {"affinity_w": float("inf")}):
        with pytest.raises(pv.PvError):
            pv.output_stage(plan, e, d, pv.output_params(**kw))
    with pytest.raises(pv.PvError):
        pv.output_stage(plan, e, d[:, :6])
    plan.close()
