"""GPU tests of the library's memory handling around a user's streams and captures."""
import threading

import numpy as np
import pytest
import torch

import paper_2506_20043_amd as pv
from paper_2506_20043_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return pv.Context(0)


def _set(ctx, seed, n=1):
    g = np.random.default_rng(seed)
    rx, rt = S.receptor(g, 800, 24.0)
    return pv.build_grids(ctx, rx, rt, S.boxes(g, n, 14.0, 14.0, 24.0, centred=True))


def _poses(ctx, B=64):
    g = np.random.default_rng(5)
    ligs = pv.Ligands(ctx, [S.tree_ligand(g, 20, 4)])
    z = torch.zeros(B, dtype=torch.int32, device="cuda")
    return ligs, z, torch.from_numpy(S.poses(g, B, np.full(3, 8.0), np.full(3, 16.0), 4).astype(np.float32)).cuda()


def test_grids_freed_while_another_thread_captures(ctx):
    """A grid set freed by another thread leaves a thread-local capture whole: its replays equal the eager result."""
    grids, other = _set(ctx, 1), _set(ctx, 2)
    ligs, z, dof = _poses(ctx)
    want = {k: v.clone() for k, v in pv.score_grad(ctx, grids, ligs, z, z, dof).items()}
    torch.cuda.synchronize()
    s, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        graph.capture_begin(capture_error_mode="thread_local")
        out = pv.score_grad(ctx, grids, ligs, z, z, dof)
        t = threading.Thread(target=other.close)
        t.start()
        t.join()
        graph.capture_end()
    for _ in range(3):
        for v in out.values():
            v.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in want:
            assert torch.equal(out[k], want[k]), k


def test_freed_maps_are_not_reused_while_a_stream_reads_them(ctx):
    """Maps freed while a dock on another stream still reads them, and a build of the same size at once: the dock's
    results are those of an undisturbed one."""
    g = np.random.default_rng(3)
    ligs = pv.Ligands(ctx, [S.tree_ligand(g, 30, 6)])
    p = pv.dock_params(chains=16, steps=100, seed=9)
    s = torch.cuda.Stream()

    def dock(after):
        grids = _set(ctx, 4)
        plan = pv.Plan(ctx, grids, ligs, [(0, 0)], p)
        plan.outputs()
        torch.cuda.synchronize()
        out = plan.run(stream=s)
        after(grids)
        torch.cuda.synchronize()
        return {k: out[k].clone() for k in ("chain_best_e", "chain_best_dof", "chain_evals")}

    want = dock(lambda grids: None)
    built = []

    def free_and_build(grids):
        grids.close()
        built.append(_set(ctx, 6))

    got = dock(free_and_build)
    for k in want:
        assert torch.equal(got[k], want[k]), k


def test_gradient_scaling_of_more_values_than_a_launch_has_threads(ctx):
    """2^32 + 2^20 values (17 GB, in place): rows at both ends and where a thread's second and third round begin."""
    g = np.random.default_rng(7)
    ligs = pv.Ligands(ctx, [S.tree_ligand(g, 12, 2)])
    row, B = 1 << 20, 4097
    grad = torch.ones((B, row), device="cuda")
    lig = torch.zeros(B, dtype=torch.int32, device="cuda")
    scale = torch.arange(2, B + 2, dtype=torch.float32, device="cuda")
    st = pv.lib().pv_scale_grad(ctx.h, ligs.h, B, lig.data_ptr(), grad.data_ptr(), row, 0, scale.data_ptr(), grad.data_ptr(),
                                torch.cuda.current_stream().cuda_stream)
    assert st == 0, pv.lib().pv_last_error()
    own = 7 + ligs.max_tors
    assert torch.equal(grad[:, :own], scale[:, None].expand(B, own))
    for b in (0, 1, 2047, 2048, 2049, 4095, 4096):
        assert bool((grad[b, own:] == 1).all()), b


def test_map_build_of_more_than_one_launch(ctx):
    """1.1 million tiles (9 GB of maps), two launches: the first box, the one that both launches work on and the last
    equal their own builds."""
    g = np.random.default_rng(8)
    rx, rt = S.receptor(g, 300, 90.0)
    boxes = [(g.uniform(30.0, 60.0, 3), np.array([239.0, 251.0, 275.0]) * 0.375, 0.375) for _ in range(17)]
    many = pv.build_grids(ctx, rx, rt, boxes)
    for b in (0, 16):   # 65,205 tiles a box: box 16 begins at tile 1,043,280, before the 1,048,576th
        one = pv.build_grids(ctx, rx, rt, [boxes[b]])
        assert torch.equal(many.maps(b), one.maps(0)), b
        one.close()
    many.close()
