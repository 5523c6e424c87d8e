"""GPU parity of score + analytic gradient (Eq. qvina_eq_3 and the chain rule
through the torsion tree of Eq. qvina_eq_1) against the oracle, on the tiny
configuration, on the full 16,384-pose differentiation workload (sampled),
on degenerate ligands and poses, and through the autograd Function."""
import numpy as np
import pytest

from gpu_util import KINK, cpu_dof, e_tol, g_ok, g_tol, near_kink
from paper_2506_20043_amd import synth as S

pytestmark = pytest.mark.gpu
KAPPA = 10.0


@pytest.fixture(scope="module")
def pv_ctx():
    import paper_2506_20043_amd as pv
    return pv.Context(0)


class Setup:
    def __init__(self, oracle, pv_ctx, rx, rt, boxes, mols):
        import paper_2506_20043_amd as pv
        self.grids = pv.build_grids(pv_ctx, rx, rt, boxes, penalty_slope=KAPPA)
        self.ligs = pv.Ligands(pv_ctx, mols)
        self.og = [oracle.Grid.build(rx, rt, b.center.astype(np.float64), b.size.astype(np.float64), b.spacing,
                                     kappa=KAPPA) for b in boxes]
        self.ol = [oracle.Ligand(m.xyz, m.types, m.bonds, m.rotatable) for m in mols]
        self.mols, self.boxes, self.ctx = mols, boxes, pv_ctx

    def lohi(self, b):
        G = self.og[b]
        return G.origin.astype(np.float64), G.origin + G.h * (G.dims - 1)


def compare(st, lig, box, dof, out, idx, max_excused=0.05):
    """Compares GPU outputs at pose rows idx with the oracle; returns the
    number of gradient mismatches excused by a nearby kink."""
    e = out["energy"].cpu().numpy()
    parts = out["e_parts"].cpu().numpy() if "e_parts" in out else None
    gd = out["grad_dof"].cpu().numpy()
    xyz = out["xyz"].cpu().numpy() if "xyz" in out else None
    gx = out["grad_xyz"].cpu().numpy() if "grad_xyz" in out else None
    excused = 0
    for b in idx:
        L, G = st.ol[lig[b]], st.og[box[b]]
        r = L.score_grad(G, cpu_dof(dof[b, :L.ndof]))
        slack = 0.01 if r["min_cut"] < KINK else 0.0
        assert abs(e[b] - r["e"]) <= e_tol(r["e"]) + slack, (b, e[b], r["e"])
        if parts is not None:
            assert abs(parts[b, 0] - r["e_inter"]) <= e_tol(r["e_inter"]), (b, parts[b], r["e_inter"])
            assert abs(parts[b, 1] - r["e_intra"]) <= e_tol(r["e_intra"]) + slack, (b, parts[b], r["e_intra"])
        if xyz is not None:
            assert np.abs(xyz[b, :L.n_atoms] - r["xyz"]).max() <= 1e-4, b
        assert np.all(gd[b, L.ndof:] == 0.0)
        gref = r["grad_dof"]
        ok = g_ok(gd[b, :L.ndof], gref, dof=True)
        if gx is not None:
            ok = ok and g_ok(gx[b, :L.n_atoms], r["grad_xyz"])
        if not ok:
            rd = np.abs(gd[b, :L.ndof] - gref) / g_tol(gref, dof=True)
            k = int(np.argmax(rd))
            msg = (b, "dof", k, float(gd[b, k]), float(gref[k]), float(rd[k]))
            if gx is not None:
                rx = np.abs(gx[b, :L.n_atoms] - r["grad_xyz"]) / g_tol(r["grad_xyz"])
                msg += ("xyz worst ratio", float(rx.max()))
            assert near_kink(r), msg
            excused += 1
    assert excused <= max_excused * len(idx), (excused, len(idx))
    return excused


def test_tiny_config_poses(oracle, pv_ctx):
    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    mols = S.make_ligands(cfg)
    st = Setup(oracle, pv_ctx, rx, rt, bxs, mols)
    g = np.random.default_rng(0)
    lo, hi = st.lohi(0)
    B = 300
    dof = S.poses(g, B, lo - 1.0, hi + 1.0, st.ol[0].n_tors)  # some poses leave the box
    z = np.zeros(B, np.int32)
    out = pv.score_grad(pv_ctx, st.grids, st.ligs, z, z, dof, parts=True, xyz=True)
    compare(st, z, z, dof, out, range(B))


def test_differentiation_workload_full_size(oracle, pv_ctx):
    """16,384 poses of 64 ligands (40 atoms, 10 torsions) in one 24 A pocket,
    the launch the benchmark times; the oracle checks a sample."""
    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["differentiation"]
    rx, rt, bxs = S.make_receptor(cfg)
    mols = S.make_ligands(cfg)
    st = Setup(oracle, pv_ctx, rx, rt, bxs[:1], mols)
    g = S.rng(cfg.index, S.STREAM_POSES)
    lo, hi = st.lohi(0)
    per = cfg.n_poses // cfg.n_ligands
    dof = S.poses(g, cfg.n_poses, lo, hi, 10)
    lig = np.repeat(np.arange(cfg.n_ligands, dtype=np.int32), per)
    box = np.zeros(cfg.n_poses, np.int32)
    out = pv.score_grad(pv_ctx, st.grids, st.ligs, lig, box, dof, parts=True)
    assert np.isfinite(out["energy"].cpu().numpy()).all()
    idx = np.random.default_rng(1).choice(cfg.n_poses, 400, replace=False)
    compare(st, lig, box, dof, out, np.sort(idx))


def test_degenerate_ligands(oracle, pv_ctx):
    """One atom, no torsion, and the largest ligand (128 atoms, 32 torsions)."""
    import paper_2506_20043_amd as pv
    g = np.random.default_rng(2)
    rx, rt = S.receptor(g, 1500, 40.0)
    box = S.Box(np.full(3, 20.0, np.float32), np.full(3, 30.0, np.float32), 0.375)
    one = S.Molecule(np.zeros((1, 3)), np.array([4], np.int32), np.zeros((0, 2), np.int32), np.zeros(0, np.uint8))
    rigid = S.tree_ligand(g, 12, 0)
    big = S.tree_ligand(g, 128, 32)
    mols = [one, rigid, big]
    st = Setup(oracle, pv_ctx, rx, rt, [box], mols)
    lo, hi = st.lohi(0)
    B = 60
    lig = np.repeat(np.arange(3, dtype=np.int32), B // 3)
    dof = np.zeros((B, 7 + 32), np.float32)
    for b in range(B):
        nt = st.ol[lig[b]].n_tors
        dof[b, :7 + nt] = S.poses(g, 1, lo + 2, hi - 2, nt)[0]
    out = pv.score_grad(pv_ctx, st.grids, st.ligs, lig, np.zeros(B, np.int32), dof, parts=True, xyz=True)
    compare(st, lig, np.zeros(B, np.int32), dof, out, range(B), max_excused=0.2)
    # rows past each pose's atoms come back zero, not uninitialised
    xyz, gx = out["xyz"].cpu().numpy(), out["grad_xyz"].cpu().numpy()
    for b in range(B):
        n = st.ol[lig[b]].n_atoms
        assert np.all(xyz[b, n:] == 0.0) and np.all(gx[b, n:] == 0.0), b


def test_invalid_rows_and_empty_batch(oracle, pv_ctx):
    import paper_2506_20043_amd as pv
    g = np.random.default_rng(3)
    rx, rt = S.receptor(g, 300, 20.0)
    box = S.Box(np.full(3, 10.0, np.float32), np.full(3, 12.0, np.float32), 0.375)
    mol = S.tree_ligand(g, 10, 2)
    st = Setup(oracle, pv_ctx, rx, rt, [box], [mol])
    dof = np.tile(np.array([10, 10, 10, 1, 0, 0, 0, 0.1, 0.2], np.float32), (4, 1))
    dof[3, 3:7] = 0.0   # zero quaternion
    out = pv.score_grad(pv_ctx, st.grids, st.ligs, [0, 5, 0, 0], [0, 0, -1, 0], dof, xyz=True)
    e = out["energy"].cpu().numpy()
    assert np.isfinite(e[0]) and np.isnan(e[1]) and np.isnan(e[2]) and np.isnan(e[3])
    assert np.isnan(out["grad_dof"].cpu().numpy()[1]).all()
    # out-of-range rows: NaN coordinates and coordinate gradients
    for k in ("xyz", "grad_xyz"):
        v = out[k].cpu().numpy()
        assert np.isnan(v[1]).all() and np.isnan(v[2]).all() and np.isfinite(v[0]).all(), k
    empty = pv.score_grad(pv_ctx, st.grids, st.ligs, np.zeros(0, np.int32), np.zeros(0, np.int32),
                          np.zeros((0, 9), np.float32))
    assert empty["energy"].numel() == 0
    with pytest.raises(pv.PvError, match="dof_stride"):
        pv.score_grad(pv_ctx, st.grids, st.ligs, [0], [0], np.zeros((1, 8), np.float32))


def test_score_on_coordinates(oracle, pv_ctx):
    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    mols = S.make_ligands(S.CONFIGS["uneven_batch"], count=6)
    st = Setup(oracle, pv_ctx, rx, rt, bxs, mols)
    g = np.random.default_rng(4)
    lo, hi = st.lohi(0)
    B = 60
    lig = np.arange(B, dtype=np.int32) % 6
    ma = st.ligs.max_atoms
    xyz = np.zeros((B, ma, 3), np.float32)
    for b in range(B):
        L = st.ol[lig[b]]
        d = S.poses(g, 1, lo, hi, L.n_tors)[0]
        xyz[b, :L.n_atoms] = L.fk(d.astype(np.float64)).astype(np.float32)
    out = pv.score_grad_xyz(pv_ctx, st.grids, st.ligs, lig, np.zeros(B, np.int32), xyz, parts=True)
    e = out["energy"].cpu().numpy()
    gx = out["grad_xyz"].cpu().numpy()
    excused = 0
    for b in range(B):
        L = st.ol[lig[b]]
        r = L.score_xyz(st.og[0], xyz[b, :L.n_atoms].astype(np.float64))
        slack = 0.01 if r["min_cut"] < KINK else 0.0
        assert abs(e[b] - r["e"]) <= e_tol(r["e"]) + slack
        if not g_ok(gx[b, :L.n_atoms], r["grad_xyz"]):
            assert near_kink(r), b
            excused += 1
    assert excused <= B // 10


def test_autograd_backward(oracle, pv_ctx):
    """ScoreGrad's backward equals grad_energy times the gradient kernel's
    output, and both agree with central differences (h = 1e-4) of the oracle."""
    import torch

    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    mols = S.make_ligands(cfg)
    st = Setup(oracle, pv_ctx, rx, rt, bxs, mols)
    g = np.random.default_rng(5)
    lo, hi = st.lohi(0)
    B = 64
    L = st.ol[0]
    dof_np = S.poses(g, B, lo + 2, hi - 2, L.n_tors)
    z = torch.zeros(B, dtype=torch.int32, device="cuda")
    handles = (pv_ctx, st.grids, st.ligs, z, z)
    dof = torch.tensor(dof_np, device="cuda", requires_grad=True)
    e = pv.ScoreGrad.apply(dof, handles)
    w = torch.tensor(g.normal(size=B), dtype=torch.float32, device="cuda")
    (e * w).sum().backward()
    grad = dof.grad.cpu().numpy()
    plain = pv.score_grad(pv_ctx, st.grids, st.ligs, z, z, dof_np)["grad_dof"].cpu().numpy()
    wn = w.cpu().numpy()
    np.testing.assert_allclose(grad, plain * wn[:, None], rtol=1e-6, atol=1e-6)
    checked = 0
    for b in range(B):
        x = dof_np[b].astype(np.float64)
        r = L.score_grad(st.og[0], x)
        if near_kink(r):
            continue
        h = 1e-4
        fd = np.zeros(L.ndof)
        for i in range(L.ndof):
            xp, xm = x.copy(), x.copy()
            xp[i] += h
            xm[i] -= h
            fd[i] = (L.score_grad(st.og[0], xp)["e"] - L.score_grad(st.og[0], xm)["e"]) / (2 * h)
        # a difference quotient may straddle a cell face; skip those rows
        fd_tol = 1e-3 * (1 + np.abs(r["grad_dof"]).max())
        if np.abs(fd - r["grad_dof"]).max() > fd_tol:
            continue
        # against the quotient at its own accuracy (its truncation error is
        # O(h^2)), and against the oracle's analytic gradient at parity
        assert np.abs(plain[b] - fd).max() <= 2 * fd_tol, b
        assert g_ok(plain[b], r["grad_dof"], dof=True), b
        checked += 1
    assert checked >= B // 2
    # coordinates form
    xyz = torch.tensor(np.stack([L.fk(d.astype(np.float64)) for d in dof_np]).astype(np.float32), device="cuda",
                       requires_grad=True)
    ex = pv.ScoreGradXYZ.apply(xyz, handles)
    ex.sum().backward()
    ref = pv.score_grad(pv_ctx, st.grids, st.ligs, z, z, dof_np, xyz=True)["grad_xyz"].cpu().numpy()
    np.testing.assert_allclose(xyz.grad.cpu().numpy(), ref[:, :L.n_atoms], rtol=1e-3, atol=1e-3)


def test_fma_peak_aid(pv_ctx):
    """The measurement aid behind the bench's measured FP32 rate: one value
    per thread, finite and the same on every call; bad arguments rejected."""
    import torch

    import paper_2506_20043_amd as pv
    out = torch.empty(4 * 256, dtype=torch.float32, device="cuda")
    flops = pv.fma_peak(pv_ctx, 8, out)
    assert flops == 2 * 16 * 8 * 1024
    a = out.cpu().clone()
    pv.fma_peak(pv_ctx, 8, out)
    assert torch.isfinite(a).all() and torch.equal(a, out.cpu())
    with pytest.raises(pv.PvError):
        pv.fma_peak(pv_ctx, 0, out)
    with pytest.raises(pv.PvError):
        pv.fma_peak(pv_ctx, 8, out[:100])


def test_ring_ligands_score_and_gradient(oracle, pv_ctx):
    """Ligands with rigid six-membered rings (rings inside fragments,
    torsions on bridges): score and gradient of random poses against the
    oracle, with one atom per lane (ligands of 20 and 36 atoms) and two (70
    atoms): the kernel variant follows the ligand set's largest ligand."""
    import paper_2506_20043_amd as pv
    g = np.random.default_rng(23)
    rx, rt = S.receptor(g, 2000, 36.0)
    box = S.Box(np.full(3, 18.0, np.float32), np.full(3, 24.0, np.float32), 0.375)
    for mols in ([S.ring_ligand(g, 20, 4, 2), S.ring_ligand(g, 36, 7, 3)], [S.ring_ligand(g, 70, 10, 4)]):
        st = Setup(oracle, pv_ctx, rx, rt, [box], mols)
        lo, hi = st.lohi(0)
        B = 120
        lig = np.arange(B, dtype=np.int32) % len(mols)
        dof = np.zeros((B, st.ligs.dof_stride), np.float32)
        for b in range(B):
            nt = st.ol[lig[b]].n_tors
            dof[b, :7 + nt] = S.poses(g, 1, lo + 2, hi - 2, nt)[0]
        z = np.zeros(B, np.int32)
        out = pv.score_grad(pv_ctx, st.grids, st.ligs, lig, z, dof, parts=True, xyz=True)
        compare(st, lig, z, dof, out, range(B))


@pytest.mark.parametrize("of_xyz", [False, True])
def test_autograd_scaling_matches_the_kernel(pv_ctx, of_xyz):
    """The backward scales the gradient that the forward kept: bit for bit the score kernel's own gradient with the
    upstream factors as grad_energy, for ragged ligands, poses of no ligand or box, zero, infinite and NaN factors; the
    energy alone (no gradient wanted) is the same too, and an input changed in place before the backward is refused."""
    import torch

    import paper_2506_20043_amd as pv
    cfg = S.CONFIGS["tiny"]
    rx, rt, bxs = S.make_receptor(cfg)
    g = np.random.default_rng(31)
    mols = [S.tree_ligand(g, n, t) for n, t in ((20, 4), (3, 0), (40, 9), (70, 12))]
    grids, ligs = pv.build_grids(pv_ctx, rx, rt, bxs[:1]), pv.Ligands(pv_ctx, mols)
    B = 203
    lig = torch.tensor(g.integers(0, 4, B), dtype=torch.int32, device="cuda")
    box = torch.zeros(B, dtype=torch.int32, device="cuda")
    lig[5], lig[6], box[7] = -1, 4, 1
    x = torch.tensor(S.poses(g, B, 6.0, 24.0, ligs.max_tors + 2), device="cuda")
    if of_xyz:
        x = pv.score_grad(pv_ctx, grids, ligs, lig, box, x, xyz=True)["xyz"].nan_to_num(5.0)
    w = torch.tensor(g.normal(size=B), dtype=torch.float32, device="cuda")
    w[:5] = torch.tensor([0.0, float("inf"), -float("inf"), float("nan"), 1.0])
    score = pv.score_grad_xyz if of_xyz else pv.score_grad
    ref = score(pv_ctx, grids, ligs, lig, box, x, grad_energy=w)
    fn = pv.ScoreGradXYZ if of_xyz else pv.ScoreGrad
    x.requires_grad_(True)
    e = fn.apply(x, (pv_ctx, grids, ligs, lig, box))
    (got,) = torch.autograd.grad(e, x, w, retain_graph=True)
    want = ref["grad_xyz" if of_xyz else "grad_dof"]
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy(), equal_nan=True)
    assert np.array_equal(e.detach().cpu().numpy(), ref["energy"].cpu().numpy(), equal_nan=True)
    with torch.no_grad():
        alone = fn.apply(x, (pv_ctx, grids, ligs, lig, box))
        assert np.array_equal(alone.cpu().numpy(), ref["energy"].cpu().numpy(), equal_nan=True)
        x.add_(1.0)
    with pytest.raises(RuntimeError):
        torch.autograd.grad(e, x, w)


@pytest.mark.parametrize("n", [1, 2049, 13000])
def test_ragged_batches_equal_their_pieces(pv_ctx, n):
    """Ligands of very different sizes run shorter runs of poses per wave: fewer poses than waves, one past them, and
    more than six per slot give what pieces of 500 poses give, bit for bit."""
    import torch

    import paper_2506_20043_amd as pv
    rx, rt, bxs = S.make_receptor(S.CONFIGS["tiny"])
    g = np.random.default_rng(13)
    mols = [S.tree_ligand(g, k, t) for k, t in ((70, 10), (8, 1), (20, 4), (12, 2), (33, 6))]
    grids, ligs = pv.build_grids(pv_ctx, rx, rt, bxs[:1]), pv.Ligands(pv_ctx, mols)
    lig = torch.tensor(g.integers(0, 5, n), dtype=torch.int32, device="cuda")
    box = torch.zeros(n, dtype=torch.int32, device="cuda")
    dof = torch.tensor(S.poses(g, n, 6.0, 24.0, ligs.max_tors), device="cuda")
    whole = pv.score_grad(pv_ctx, grids, ligs, lig, box, dof, parts=True, xyz=True)
    for a in range(0, n, 500):
        part = pv.score_grad(pv_ctx, grids, ligs, lig[a:a + 500], box[a:a + 500], dof[a:a + 500], parts=True, xyz=True)
        for k, v in part.items():
            assert torch.equal(whole[k][a:a + 500], v), k
