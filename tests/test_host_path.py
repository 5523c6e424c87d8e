"""CPU tests of the library's host code on a HIP runtime without a device
(fake_hip.cpp): allocations that fail, launches' sizes, what is called while a
stream captures."""
import ctypes as C

import pytest

import fake_hip


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = fake_hip.build(tmp_path_factory.mktemp("fake_hip"))
    return lambda scenario: fake_hip.run(so, "test_host_path", scenario.__name__)


# ---------------------------------------------------------------- memory
def recovered_allocation(f):
    """An allocation that succeeds once the kept map block is freed leaves no error
    behind: the launch after it does not report one."""
    ctx = f.context()
    f.grids(ctx).close()
    kept = f.rt.fake_used()
    assert kept >= 21 ** 3 * 32
    # room for the tables of two atoms' worth of boxes only when the block goes
    from paper_2506_20043_amd import synth as S
    import numpy as np
    f.rt.fake_memory(kept + 64)
    ligs = f.pv.Ligands(ctx, [S.tree_ligand(np.random.default_rng(0), 12, 2)])
    assert f.rt.fake_used() < kept
    f.rt.fake_memory(1 << 40)
    assert f.lib.pv_fma_peak(ctx.h, 1, 1 << 20, 256, None) == 0, f.lib.pv_last_error()
    ligs.close()


def failed_allocation(f):
    """Nor does one that fails: once there is room the same call succeeds."""
    ctx = f.context()
    f.rt.fake_memory(1000)
    assert f.grids(ctx) == -3
    f.rt.fake_memory(1 << 40)
    g = f.grids(ctx)
    assert g != -4, f.lib.pv_last_error()
    g.close()


@pytest.mark.parametrize("scenario", [recovered_allocation, failed_allocation], ids=lambda s: s.__name__)
def test_allocation_errors_are_not_left_behind(fake, scenario):
    fake(scenario)


def kept_block(f):
    """Freed maps up to 1 GiB are kept until pv_trim, a build of other sizes or the last context's end; larger ones never."""
    a, b = f.context(), f.context()
    f.grids(a).close()
    assert f.rt.fake_used() == 21 ** 3 * 32
    assert f.lib.pv_trim(a.h) == 0 and f.rt.fake_used() == 0
    assert f.lib.pv_trim(a.h) == 0                       # nothing kept
    assert f.lib.pv_trim(None) == -6
    f.grids(a).close()
    f.grids(a, boxes=[([0., 0, 0], 300.0, 1.5)]).close()   # 201^3 points, 260 MB: the smaller block goes
    assert 201 ** 3 * 32 <= f.rt.fake_used() < 201 ** 3 * 32 + 1000
    f.grids(a, boxes=[([0., 0, 0], 300.0, 1.5)] * 5).close()   # 1.3 GB
    assert f.rt.fake_used() == 0
    f.grids(a).close()
    f.lib.pv_destroy(a.h)
    assert f.rt.fake_used() > 0
    f.lib.pv_destroy(b.h)
    assert f.rt.fake_used() == 0


def test_kept_map_block(fake):
    fake(kept_block)


def current_device(f):
    """Destroying a device's last context frees its kept block and leaves the thread's current device as it is."""
    a, b = f.context(0), f.context(1)
    f.grids(b).close()
    f.lib.pv_trim(a.h)
    assert f.rt.fake_current_device() == 0 and f.rt.fake_used() > 0
    f.lib.pv_destroy(b.h)
    assert f.rt.fake_current_device() == 0 and f.rt.fake_used() == 0


def test_current_device_after_a_context_ends(fake):
    fake(current_device)


# ---------------------------------------------------------------- captures
def free_during_capture(f):
    """Freeing grids while a stream captures makes no call that waits for the device, keeps no block that the device
    may still use, and leaves no error behind."""
    ctx = f.context()
    a, b = f.grids(ctx), f.grids(ctx)
    f.rt.fake_capture(1)
    a.close()
    assert f.rt.fake_device_syncs() == 0
    assert f.lib.pv_fma_peak(ctx.h, 1, 1 << 20, 256, None) == 0, f.lib.pv_last_error()
    f.rt.fake_capture(0)
    used = f.rt.fake_used()
    c = f.grids(ctx)   # the block of `a` was not kept: this build allocates
    assert f.rt.fake_used() > used + 21 ** 3 * 32
    b.close()
    c.close()


def test_grids_freed_during_a_capture(fake):
    fake(free_during_capture)


# ---------------------------------------------------------------- launch sizes
def scale_launches(f):
    """Every number of values is launched with fewer than 2^32 threads (the runtime takes no more in a dimension)."""
    import numpy as np
    from paper_2506_20043_amd import synth as S
    ctx = f.context()
    ligs = f.pv.Ligands(ctx, [S.tree_ligand(np.random.default_rng(0), 12, 2)])
    p = 1 << 20
    for poses, row, xyz in ((1, 9, 0), (16384, 17, 0), (1 << 27, 16, 0), ((1 << 28) + 1, 16, 0), (11200000, 384, 1)):
        st = f.lib.pv_scale_grad(ctx.h, ligs.h, poses, p, p, row, xyz, p, p, None)
        assert st == 0, (poses, row, f.lib.pv_last_error())
        (k,) = f.launches("scale_grad")
        assert k[1][0] * k[2][0] >= min(poses * row, 1 << 31) and k[1][1] == k[1][2] == 1


def test_gradient_scaling_launches(fake):
    fake(scale_launches)


def grid_launches(f):
    """Map builds of up to 2^24 tiles (137 GB of maps), and around a launch's most: every tile has a workgroup, in
    whole runs of 32, in launches of at most 2^20."""
    ctx = f.context()

    def box(nx, ny, nz):
        return [0.0, 0, 0], [nx - 1.0, ny - 1.0, nz - 1.0], 1.0

    big = (240, 252, 276)                  # 15 x 63 x 69 tiles
    for sizes, tiles in (([(5, 4, 4)], 1), ([big] * 16 + [(240, 80, 28)], 16 * 65205 + 2100), ([big] * 17, 17 * 65205),
                         ([big] * 257 + [(240, 80, 260)], (1 << 24) - 31)):
        g = f.grids(ctx, boxes=[box(*s) for s in sizes])
        assert not isinstance(g, int), (tiles, f.lib.pv_last_error())
        grids = [k[1] for k in f.launches("gridmap")]
        assert all(x % 32 == 0 and x <= 1 << 20 and y == z == 1 for x, y, z in grids)
        assert all(x == 1 << 20 for x, _, _ in grids[:-1]) and tiles <= sum(x for x, _, _ in grids) < tiles + 32
        g.close()


def test_grid_map_launches(fake):
    fake(grid_launches)


# ---------------------------------------------------------------- output stage
def output_waves(f):
    """Waves per job of the output stage: eight, or as many as the LDS holds, for few jobs; for many jobs as many as keep
    every wave at work (four whatever the modes took up to 1.9 times as long as one)."""
    import numpy as np
    from paper_2506_20043_amd import synth as S
    pv, ctx = f.pv, f.context()
    grids = f.grids(ctx)
    p = 1 << 20
    for atoms, tors, jobs, modes, want in ((64, 20, 120, 20, 7), (64, 20, 1500, 5, 1), (64, 20, 6000, 3, 1), (64, 20, 1000, 20, 7),
                                           (20, 4, 5, 3, 8), (20, 4, 1000, 20, 4), (20, 4, 2000, 9, 1), (100, 20, 2000, 3, 3),
                                           (100, 20, 120, 20, 5)):
        ligs = pv.Ligands(ctx, [S.tree_ligand(np.random.default_rng(atoms * 31 + tors), atoms, tors)])
        plan = pv.Plan(ctx, grids, ligs, [(0, 0)] * jobs, pv.dock_params(chains=32))
        o, op = pv.ModesOut(p, p, p, p, p, 7 + tors), pv.output_params(modes=modes)
        f.launches()
        assert f.lib.pv_output_stage(plan.h, p, p, 7 + tors, C.byref(op), C.byref(o), None) == 0, f.lib.pv_last_error()
        (k,) = f.launches("output_kernel")
        assert k[1][0] == jobs and k[2] == (64, want, 1), (atoms, jobs, modes, k[2])


def test_output_stage_waves(fake):
    fake(output_waves)


# ---------------------------------------------------------------- surface points
def surface_launches(f):
    """Few atoms with many directions fill the chip, or take a wave per 64 directions of two atoms; many atoms take a wave
    per two."""
    import numpy as np
    ctx = f.context()
    for atoms, dirs, waves in ((20, 4096, 640), (500, 4096, 2000), (500, 1000, 2000), (1, 33, 1), (2000, 30, 1000), (8000, 4096, 4000)):
        x, t, d = np.zeros((atoms, 3), np.float32), np.zeros(atoms, np.uint8), np.ones((dirs, 3), np.float32)
        h = C.c_void_p()
        f.launches()
        assert f.lib.pv_sas_build(ctx.h, atoms, x.ctypes.data, t.ctypes.data, dirs, d.ctypes.data, 1.6, None, C.byref(h)) == 0
        (k,) = f.launches("sas_keep")
        got = (atoms + 1) // 2 * k[1][1]
        assert waves <= got <= 2 * waves, (atoms, dirs, got)
        f.lib.pv_sas_free(h)


def test_surface_launches(fake):
    fake(surface_launches)


# ---------------------------------------------------------------- helper waves
def team_sizes(f):
    """On a caller's stream teams leave room for the equal launches of other streams that fit beside a launch of one wave
    per chain, up to four (the hardware queues of a process); on the null stream all its chains are resident."""
    import numpy as np
    from paper_2506_20043_amd import synth as S
    pv, ctx = f.pv, f.context()
    grids = f.grids(ctx)
    o = pv.DockOut()
    for atoms, tors in ((20, 4), (35, 8), (60, 12)):
        ligs = pv.Ligands(ctx, [S.tree_ligand(np.random.default_rng(atoms), atoms, tors)])
        for stream, side in ((None, 1), (0x77770, 4)):
            seen = set()
            for chains in (1, 8, 40, 160, 192, 193, 240, 320, 384, 385, 500, 750, 1280, 1500):
                plan = pv.Plan(ctx, grids, ligs, [(0, 0)], pv.dock_params(chains=chains))
                plan.set_schedule(0, pv.VARIANT_SLOTS, 0)
                n, one = C.c_int32(), plan.schedule()["per_cu"] * 256
                assert f.lib.pv_plan_waves(plan.h, 0, stream, C.byref(n)) == 0
                w = n.value
                # twelve waves per CU at these kernels' registers, less where the LDS holds fewer
                assert 12 // w * 256 >= chains * min(side, one // chains) or w == 1, (atoms, chains, w)
                f.launches()
                assert f.lib.pv_dock_run(plan.h, C.byref(o), stream) == 0
                assert [k[2] for k in f.launches("dock_kernel")] == [(64, w, 1)]
                seen.add(w)
                plan.close()
            assert seen >= ({4, 2} if atoms < 60 else {4}), (atoms, seen)
        ligs.close()


def test_teams_leave_room_for_other_streams(fake):
    fake(team_sizes)


# ---------------------------------------------------------------- size classes
def classes_on_streams(f):
    """Two size classes run side by side on the null stream and where they fill the GPU; smaller launches on a stream of
    the caller's run one after the other on it (its hardware queue is not the only one that others may wait for)."""
    import numpy as np
    from paper_2506_20043_amd import synth as S
    pv, ctx, g = f.pv, f.context(), np.random.default_rng(3)
    grids = f.grids(ctx)
    ligs = pv.Ligands(ctx, [S.tree_ligand(g, 30, 5), S.tree_ligand(g, 90, 8)])
    o = pv.DockOut()
    for flags in (0, pv.PV_DOCK_GRAPH):
        for jobs, stream, beside in ((3, None, True), (3, 0x77770, False), (200, None, True), (200, 0x77770, True)):
            plan = pv.Plan(ctx, grids, ligs, [(0, 0), (1, 0)] * jobs, pv.dock_params(chains=16, flags=flags))
            f.launches()
            assert f.lib.pv_dock_run(plan.h, C.byref(o), stream) == 0, f.lib.pv_last_error()
            streams = [k[4] for k in f.launches("dock_kernel")]
            assert len(streams) == 2 and (streams[0] != streams[1]) == beside, (flags, jobs, stream, streams)
            if not flags:
                assert streams[0] == (stream or 0)
            plan.close()


def test_size_classes_beside_other_streams(fake):
    fake(classes_on_streams)


# ---------------------------------------------------------------- autotuner
def _tune(f, plan, repeats=1):
    """(group, variant, workgroups, cached) of every candidate, and the dock launches."""
    pv = f.pv
    res, n = (pv.TuneResult * 64)(), C.c_int32()
    f.launches()
    assert f.lib.pv_dock_autotune(plan.h, 2, repeats, None, res, 64, C.byref(n)) == 0, f.lib.pv_last_error()
    return [(r.group, r.variant, r.workgroups, r.cached) for r in res[:n.value]], f.launches("dock_kernel")


def _tune_plans(f):
    """A plan of one size class, and one with the same class and a larger one."""
    import numpy as np
    from paper_2506_20043_amd import synth as S
    g, ctx = np.random.default_rng(3), f.context()
    grids = f.grids(ctx)
    ligs = f.pv.Ligands(ctx, [S.tree_ligand(g, 30, 5), S.tree_ligand(g, 90, 8)])
    p = f.pv.dock_params(chains=16)
    return [f.pv.Plan(ctx, grids, ligs, jobs, p) for jobs in ([(0, 0)] * 4, [(0, 0)] * 4, [(0, 0)] * 4 + [(1, 0)] * 3)]


def tuned_choices(f):
    """A class's remembered schedule is not taken where another class runs beside it, which decides about its helper
    waves; one of an equal plan is."""
    one, same, two = _tune_plans(f)
    assert all(r[3] == 0 for r in _tune(f, one)[0])
    assert [r[3] for r in _tune(f, same)[0]] == [1]
    res, _ = _tune(f, two)
    assert {r[0] for r in res} == {0, 1} and all(r[3] == 0 for r in res), res
    assert [r[3] for r in _tune(f, two)[0]] == [1, 1]


def tuned_side_by_side(f):
    """Every candidate of a plan of two classes is timed as the plan runs: both classes' launches, on two streams."""
    one, _, two = _tune_plans(f)
    for plan, classes in ((one, 1), (two, 2)):
        res, launches = _tune(f, plan, repeats=3)
        assert len(launches) == 3 * classes * len(res)
        for k in range(0, len(launches), classes):
            assert len({x[4] for x in launches[k:k + classes]}) == classes


@pytest.mark.parametrize("scenario", [tuned_choices, tuned_side_by_side], ids=lambda s: s.__name__)
def test_autotuner(fake, scenario):
    fake(scenario)
