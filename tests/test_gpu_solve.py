"""Frame-solve parity on the GPU: the whole flip-flop / CG / hierarchy
schedule through vd_solve_frame against the oracle's replica mode (the same
Jacobi-PCG algorithm and counts in float64).  Gates: final energy within
1e-4 relative, node positions within 1e-3 of the finest spacing."""

import numpy as np
import pytest

import oracle
from synth import make_config0, make_config1, make_tiny, random_rotation
from synth.scenes import make_identity_scene, make_rigid_scene

from helpers import grids_of, make_lattice, rel_err, rotation_angle

pytestmark = pytest.mark.gpu


def _check_against_oracle(scene, lat_kw=None, e_tol=1e-4, x_tol=1e-3, r_tol=1e-4):
    """Gates: float32 mode as the target states (1e-4 energy, 1e-3 spacing)
    and 1e-4 rad (measured up to 2.2e-6 rad at 64^3); float64 mode through
    the float64 state export at 1e-12 / 1e-10 / 1e-10 rad (measured 4e-16,
    5e-15 and 8e-15: rounding-order differences that truncated CG may
    amplify by orders of magnitude)."""
    if (lat_kw or {}).get("precision") == "fp64":
        e_tol, x_tol, r_tol = 1e-12, 1e-10, 1e-10
    ref = oracle.solve_frame(scene)
    lat = make_lattice(scene, **(lat_kw or {}))
    rep = lat.solve_frame(report=True)
    assert not rep["bits"] & 16  # no grid-barrier timeout in a persistent CG loop
    pos, rot = lat.get_state64()
    h = scene.spec.spacing
    dx = np.abs(pos - ref["t"]).max() / h
    e_gpu, e_ref = rep["energy"], np.asarray(ref["energy"])
    e_rel = abs(e_gpu[0] / e_ref[0] - 1.0)
    dr = rotation_angle(rot, ref["R"]).max()
    print(f"E rel {e_rel:.2e}, max |dt|/h {dx:.2e}, max rotation angle {dr:.2e} rad")
    assert e_rel < e_tol, (e_gpu, e_ref)
    assert dx < x_tol, dx
    assert dr < r_tol, dr
    np.testing.assert_allclose(lat.get_energy(), e_gpu, rtol=1e-12)
    # the float32 export is the float64 state rounded
    pos32, rot32 = lat.get_state()
    np.testing.assert_array_equal(pos32, pos.astype(np.float32))
    np.testing.assert_array_equal(rot32, rot.astype(np.float32))
    return lat, rep, ref


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_cfg0_matches_replica(precision):
    _check_against_oracle(make_config0(0), {"precision": precision})


@pytest.mark.parametrize("seed", [1, 2])
def test_ragged_multilevel_matches_replica(seed):
    scene = make_tiny(seed=seed, dims=(19, 14, 10), num_levels=3, gn=3, pcg=8, n_dense=800,
                      n_sparse=30, spacing=0.7, origin=(0.5, -2.0, 1.0))
    _check_against_oracle(scene)


@pytest.mark.parametrize("dims,levels,precision", [((2, 2, 2), 1, "fp32"), ((2, 2, 2), 1, "fp64"),
                                                  ((3, 3, 3), 2, "fp32"), ((3, 4, 5), 2, "fp64")])
def test_smallest_lattices_match_replica(dims, levels, precision):
    """The smallest lattices (one cell per axis, or a 2-node coarse level
    under a 3-node one): one tile per level, the persistent CG loop with a
    single workgroup, every sample in the last cell of each axis."""
    scene = make_tiny(seed=40 + sum(dims), dims=dims, num_levels=levels, gn=3, pcg=6,
                      n_dense=60, n_sparse=4, spacing=0.8, origin=(0.2, -0.1, 0.3))
    _check_against_oracle(scene, {"precision": precision})


def test_cfg1_matches_replica():
    """The 64^3, 3-level x 8 GN x 20 PCG frame the benchmark times."""
    lat, rep, ref = _check_against_oracle(make_config1(0))
    assert rep["bits"] & 1 == 0  # no CG guard hits on a well-posed frame


def test_graph_replay_equals_eager():
    scene = make_config0(1)
    eager = make_lattice(scene)
    graph = make_lattice(scene, graph=True)
    for k in range(3):
        e1 = eager.solve_frame(reset=True, report=True)["energy"]
        e2 = graph.solve_frame(reset=True, report=True)["energy"]
        np.testing.assert_array_equal(e1, e2)
    np.testing.assert_array_equal(eager.get_state()[0], graph.get_state()[0])


def test_deterministic_rerun_and_resume():
    scene = make_config0(2)
    a = make_lattice(scene)
    a.solve_frame()
    pos_a, rot_a = a.get_state()
    a.solve_frame()
    pos_a2, _ = a.get_state()
    # resume from a checkpoint of the first frame in a fresh handle: the
    # checkpoint holds float32 positions, so the resumed frame agrees to the
    # rounding of those positions
    b = make_lattice(scene)
    b.set_state(pos_a, rot_a)
    b.solve_frame()
    np.testing.assert_allclose(b.get_state()[0], pos_a2, rtol=0, atol=1e-5 * scene.spec.spacing)
    # a fresh handle from rest reproduces the first frame bit for bit
    c = make_lattice(scene)
    c.solve_frame()
    np.testing.assert_array_equal(c.get_state()[0], pos_a)


def test_trace_is_monotone():
    scene = make_config0(3)
    lat = make_lattice(scene, trace=True)
    rep = lat.solve_frame(report=True)
    tr = rep["trace"]
    assert tr.size == 2 * scene.spec.gn_iters[0]
    assert np.all(np.diff(tr) <= 1e-6 * tr[:-1])
    trace_ref = []
    oracle.solve_frame(scene, trace=trace_ref)
    np.testing.assert_allclose(tr, [e for (_, _, e) in trace_ref], rtol=1e-4)


@pytest.mark.parametrize("levels", [1, 3])
def test_rigid_fixed_point(levels):
    rng = np.random.default_rng(10 + levels)
    base = make_tiny(seed=10 + levels, dims=(17, 12, 9), num_levels=levels, gn=2, pcg=6,
                     n_dense=300, n_sparse=8)
    Q = random_rotation(rng)
    c = rng.normal(size=3)
    scene = make_rigid_scene(base, Q, c)
    fin = grids_of(scene)[-1]
    t0 = (fin.rest_positions() @ Q.T + c).astype(np.float32)
    R0 = np.broadcast_to(Q, (fin.n, 3, 3)).astype(np.float32)
    lat = make_lattice(scene)
    lat.set_state(t0, R0)
    e0 = lat.get_energy()
    lat.solve_frame()
    pos, rot = lat.get_state()
    assert np.abs(pos - t0).max() < 1e-4 * scene.spec.spacing * 10
    assert rotation_angle(rot, R0).max() < 1e-4
    assert lat.get_energy()[0] <= max(e0[0], 1e-9) * 1.01


@pytest.mark.parametrize("levels", [1, 3])
def test_identity_stays_at_rest(levels):
    base = make_tiny(seed=20, dims=(9, 9, 9), num_levels=levels, n_dense=100)
    scene = make_identity_scene(base)
    lat = make_lattice(scene)
    rep = lat.solve_frame(report=True)
    pos, rot = lat.get_state()
    rest = grids_of(scene)[-1].rest_positions()
    assert np.all(np.isfinite(pos)) and np.all(np.isfinite(rot))
    assert np.abs(pos - rest).max() < 1e-5
    assert rotation_angle(rot, np.broadcast_to(np.eye(3), rot.shape)).max() < 1e-5
    assert rep["energy"][0] < 1e-8


def test_validation_errors_leave_handle_unchanged():
    from paper_1603_08161_amd import VDError, VD_ERANGE, VD_EINVAL, VD_ESTATE
    scene = make_config0(4)
    from paper_1603_08161_amd import Lattice
    lat = Lattice.from_spec(scene.spec)
    with pytest.raises(VDError) as ei:
        lat.solve_frame()
    assert ei.value.code == VD_ESTATE
    lat.set_scene(scene)
    lat.solve_frame()
    e_ok = lat.get_energy()
    bad = scene.canon.copy()
    bad[7] = [20.0, 1.0, 1.0]
    with pytest.raises(VDError) as ei:
        lat.set_constraints(bad, scene.target, scene.normal, scene.weight,
                            scene.sparse_canon, scene.sparse_target)
    assert ei.value.code == VD_ERANGE
    nan = scene.target.copy()
    nan[3, 1] = np.nan
    with pytest.raises(VDError) as ei:
        lat.set_constraints(scene.canon, nan, scene.normal)
    assert ei.value.code == VD_EINVAL
    neg = scene.weight.copy()
    neg[0] = -1
    with pytest.raises(VDError) as ei:
        lat.set_constraints(scene.canon, scene.target, scene.normal, neg)
    assert ei.value.code == VD_EINVAL
    np.testing.assert_allclose(lat.get_energy(), e_ok, rtol=1e-12)


def test_device_tensor_inputs_match_host():
    import torch
    scene = make_config0(5)
    host = make_lattice(scene)
    host.solve_frame()
    dev = make_lattice(scene)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dev.set_constraints(t(scene.canon), t(scene.target), t(scene.normal), t(scene.weight),
                        t(scene.sparse_canon), t(scene.sparse_target))
    dev.solve_frame()
    np.testing.assert_array_equal(host.get_state()[0], dev.get_state()[0])


def test_empty_constraints():
    base = make_tiny(seed=30, dims=(6, 5, 4), n_dense=0, n_sparse=0)
    lat = make_lattice(base)
    rep = lat.solve_frame(report=True)
    pos, _ = lat.get_state()
    np.testing.assert_allclose(pos, grids_of(base)[-1].rest_positions(), atol=1e-6)
    assert rep["energy"][0] == 0.0


@pytest.mark.parametrize("tile", [1, 2, 3, 4, 5, 6, 7, 8])
def test_every_tile_kind_matches_replica(tile):
    scene = make_tiny(seed=7, dims=(37, 21, 18), num_levels=3, gn=3, pcg=8, n_dense=1500,
                      n_sparse=30, spacing=0.5, origin=(0.0, 0.0, 0.0))
    _check_against_oracle(scene, {"tiles": (tile, tile, tile)})


@pytest.mark.parametrize("tile", [1, 2, 3, 4, 5, 6, 7, 8])
def test_every_node_with_data_blocks(tile):
    """Samples in every cell, so every node carries data blocks: each tile's
    data-block work takes several rounds of its workgroup (4 to 13 by tile
    kind), and nodes near tile faces read rows whose neighbours sit in the
    halo."""
    scene = make_tiny(seed=11, dims=(24, 20, 16), num_levels=1, gn=3, pcg=8, n_dense=20000,
                      n_sparse=40, spacing=0.5, origin=(0.3, 0.1, -0.2))
    _check_against_oracle(scene, {"tiles": (tile,)})


@pytest.mark.parametrize("tile", [1, 4, 6, 7, 8])
def test_fp64_tile_kinds(tile):
    """The all-float64 mode on the larger tiles (their LDS doubles) and on a
    lattice whose every node carries data blocks."""
    scene = make_tiny(seed=12, dims=(24, 20, 16), num_levels=2, gn=2, pcg=8, n_dense=20000,
                      n_sparse=40, spacing=0.5, origin=(0.3, 0.1, -0.2))
    _check_against_oracle(scene, {"tiles": (tile, tile), "precision": "fp64"}, e_tol=1e-9,
                          x_tol=1e-5)


def test_autotuner_keeps_parity():
    scene = make_config0(6)
    ref = oracle.solve_frame(scene)
    lat = make_lattice(scene, graph=True)
    tiles, us = lat.tune(iters=5)
    from paper_1603_08161_amd._lib import VD_TILE_KINDS
    assert len(tiles) == 1 and 1 <= tiles[0] <= VD_TILE_KINDS
    assert all(u > 0 for u in us[0])
    rep = lat.solve_frame(report=True)
    assert abs(rep["energy"][0] / ref["energy"][0] - 1.0) < 1e-4


@pytest.mark.parametrize("maker,precision,graph", [(make_config0, "fp32", False),
                                                   (make_config0, "fp64", True),
                                                   (make_config1, "fp32", True)])
def test_cg_loops_match_per_iteration_launches(maker, precision, graph):
    """Three ways to launch a level's CG solve: one launch per iteration
    (VD_FLAG_ITERATIVE); the default, where a level of at most 16 tiles runs
    the solve as one persistent launch with grid barriers; and
    VD_FLAG_PERSIST, the persistent launch on levels of at most 128 tiles.
    They compute the same iterates (same operations, so equal up to
    floating-point contraction choices) and never time out."""
    from paper_1603_08161_amd import VD_REPORT_BARRIER_TIMEOUT
    scene = maker(0)
    out = {}
    for mode, kw in (("iterative", dict(iterative=True)), ("default", {}),
                     ("persistent", dict(persistent=True))):
        lat = make_lattice(scene, precision=precision, graph=graph, **kw)
        rep = lat.solve_frame(report=True)
        assert not rep["bits"] & VD_REPORT_BARRIER_TIMEOUT
        out[mode] = (rep["energy"], lat.get_state()[0])
    h = scene.spec.spacing
    tol = 1e-6 if precision == "fp32" else 1e-12
    for mode in ("default", "persistent"):
        assert abs(out[mode][0][0] / out["iterative"][0][0] - 1.0) < tol, mode
        dx = np.abs(out[mode][1].astype(np.float64) - out["iterative"][1]).max() / h
        assert dx < (1e-5 if precision == "fp32" else 1e-6), (mode, dx)


@pytest.mark.parametrize("active", [False, True])
@pytest.mark.parametrize("tile", range(1, 9))
def test_default_cg_loop_with_every_tile_kind(tile, active):
    """The persistent CG loop (the default on a 16^3 level: 2 to 16 tiles with
    every tile kind), with and without the optimised set M, against one
    launch per CG iteration; two frames in a row, so the second starts from
    the first one's barrier counters."""
    from paper_1603_08161_amd import VD_REPORT_BARRIER_TIMEOUT
    scene = make_config0(0)
    out = {}
    for iterative in (True, False):
        lat = make_lattice(scene, tiles=(tile,), iterative=iterative, active_set=active)
        for _ in range(2):
            rep = lat.solve_frame(report=True)
            assert not rep["bits"] & VD_REPORT_BARRIER_TIMEOUT
        out[iterative] = (rep["energy"], lat.get_state()[0])
    assert abs(out[False][0][0] / out[True][0][0] - 1.0) < 1e-6
    dx = np.abs(out[False][1].astype(np.float64) - out[True][1]).max() / scene.spec.spacing
    assert dx < 1e-5, dx


@pytest.mark.parametrize("seed,graph", [(1, False), (2, True), (3, False)])
def test_default_cg_loop_on_ragged_levels(seed, graph):
    """A ragged 3-level lattice whose two coarse levels (4 and 1 tiles) run
    their CG solves as persistent launches by default: the same iterates as
    one launch per CG iteration, to the last bit, eager and graph-replayed
    (a barrier that let a workgroup read a neighbour's stale halo shows up
    here as a drift of 1e-3 of the spacing)."""
    scene = make_tiny(seed=seed, dims=(19, 14, 10), num_levels=3, gn=3, pcg=8, n_dense=800,
                      n_sparse=30, spacing=0.7, origin=(0.5, -2.0, 1.0))
    out = {}
    for iterative in (True, False):
        lat = make_lattice(scene, iterative=iterative, graph=graph)
        for _ in range(2):
            rep = lat.solve_frame(reset=True, report=True)
        out[iterative] = (rep["energy"], lat.get_state()[0])
    np.testing.assert_array_equal(out[False][0], out[True][0])
    np.testing.assert_array_equal(out[False][1], out[True][1])


@pytest.mark.parametrize("tile", [4, 6, 7, 8])
def test_persistent_cg_loop_on_large_tiles(tile):
    """The persistent loop with the 1024- and 512-thread tiles on a lattice
    whose every node carries data blocks (20-40 tiles, all resident)."""
    from paper_1603_08161_amd import VD_REPORT_BARRIER_TIMEOUT
    scene = make_tiny(seed=13, dims=(24, 20, 16), num_levels=1, gn=2, pcg=8, n_dense=20000,
                      n_sparse=40, spacing=0.5, origin=(0.3, 0.1, -0.2))
    out = {}
    for persistent in (True, False):
        lat = make_lattice(scene, tiles=(tile,), persistent=persistent)
        rep = lat.solve_frame(report=True)
        assert not rep["bits"] & VD_REPORT_BARRIER_TIMEOUT
        out[persistent] = (rep["energy"], lat.get_state()[0])
    assert abs(out[True][0][0] / out[False][0][0] - 1.0) < 1e-6
    dx = np.abs(out[True][1].astype(np.float64) - out[False][1]).max() / scene.spec.spacing
    assert dx < 1e-5, dx


def test_graph_profile_events_time_the_finest_cg_and_change_nothing():
    """With graph + profile, HIP events captured in the frame time the finest
    level's CG iterations of every replay; the solve itself is unchanged."""
    scene = make_config1(0)
    plain = make_lattice(scene, graph=True)
    plain.solve_frame()
    e_plain = plain.get_energy()
    prof = make_lattice(scene, graph=True, profile=True)
    for _ in range(2):
        prof.solve_frame(reset=True)
    us, n = prof.profile()
    gn, pcg = scene.spec.gn_iters[-1], scene.spec.pcg_iters[-1]
    assert n["cg_a"] == gn * (pcg - 1)
    assert 0.5 < us["cg_a"] < 5000.0
    np.testing.assert_array_equal(prof.get_energy(), e_plain)


@pytest.mark.parametrize("tile", range(1, 9))
@pytest.mark.parametrize("precision,active", [("fp32", False), ("fp32", True), ("fp64", False)])
def test_one_launch_solves_equal_per_iteration_launches(tile, precision, active):
    """One-launch CG solves with every tile kind on a ragged lattice (remainders
    in every axis; up to 256 nodes of a tile carry data blocks, more than one
    round of the lanes), run as a gang and abandoned to the ticket counter,
    with 1, 2 and 7 iterations: the bits of one launch per iteration."""
    scene = make_tiny(seed=5, dims=(37, 11, 18), num_levels=2, gn=2, pcg=7, n_dense=3000,
                      n_sparse=20, spacing=0.6, origin=(0.2, -1.0, 0.4))
    for pcg in (1, 2, 7):
        scene.spec.pcg_iters = (pcg, pcg)
        out = {}
        for mode in ("iterative", "gang", "tickets"):
            lat = make_lattice(scene, tiles=(tile, tile), iterative=mode == "iterative",
                               precision=precision, active_set=active)
            lat.debug_abandon_loops(mode == "tickets")
            rep = lat.solve_frame(reset=True, report=True)
            assert not rep["bits"] & 16
            out[mode] = (rep["energy"], lat.get_state64()[0])
        for mode in ("gang", "tickets"):
            np.testing.assert_array_equal(out[mode][0], out["iterative"][0])
            np.testing.assert_array_equal(out[mode][1], out["iterative"][1])


@pytest.mark.parametrize("active", [False, True])
@pytest.mark.parametrize("dims", [(65, 64, 65), (81, 80, 83), (96, 96, 96)])
def test_one_launch_solves_on_large_levels(dims, active):
    """Levels that only the 16x16x8, 16x16x12 and 16x16x14 tiles cover (one node
    past the smaller kinds, remainders, the largest; with M tiles without
    unknowns, and the largest back on launches per iteration): the gang and its abandoned form give the same bits, and the
    state of one launch per iteration up to the order of the float64 sums,
    whose rounding truncated float32 CG amplifies to about 1e-6 of a spacing."""
    scene = make_tiny(seed=7, dims=dims, num_levels=1, gn=2, pcg=7,
                      n_dense=300 if active else 12000, n_sparse=20,
                      spacing=0.5, origin=(0.2, -1.0, 0.4))
    out = {}
    for mode in ("iterative", "gang", "tickets"):
        lat = make_lattice(scene, iterative=mode == "iterative", active_set=active)
        lat.debug_abandon_loops(mode == "tickets")
        rep = lat.solve_frame(reset=True, report=True)
        assert not rep["bits"] & 16
        out[mode] = (rep["energy"], lat.get_state64()[0])
    np.testing.assert_array_equal(out["tickets"][0], out["gang"][0])
    np.testing.assert_array_equal(out["tickets"][1], out["gang"][1])
    assert abs(out["gang"][0][0] / out["iterative"][0][0] - 1.0) < 1e-6
    assert np.abs(out["gang"][1] - out["iterative"][1]).max() < 1e-5 * scene.spec.spacing


@pytest.mark.parametrize("n_dense,n_sparse", [(0, 3), (1, 0), (257, 5), (3000, 40)])
def test_device_inputs_equal_host_inputs(n_dense, n_sparse):
    """Inputs in device memory, at odd float offsets: the state of host inputs,
    to the last bit, and the same errors for bad values (empty parts, one
    sample, one past a workgroup, several workgroups)."""
    import torch
    from paper_1603_08161_amd import Lattice, VDError, VD_ERANGE, VD_EINVAL
    scene = make_tiny(seed=2, dims=(12, 9, 10), n_dense=max(n_dense, 1), n_sparse=n_sparse)
    host = [scene.canon, scene.target, scene.normal, scene.weight, scene.sparse_canon,
            scene.sparse_target]
    host = [x[:n_dense] for x in host[:4]] + host[4:]

    def shifted(x):
        flat = torch.zeros(x.size + 3, device="cuda")
        flat[3:] = torch.from_numpy(np.ascontiguousarray(x)).reshape(-1).cuda()
        return flat[3:].view(x.shape)

    def solved(arrays):
        lat = Lattice.from_spec(scene.spec)
        lat.set_constraints(*[x if len(x) else None for x in arrays])
        lat.solve_frame(reset=True)
        return lat.get_state()
    ref = solved(host)
    got = solved([shifted(x) for x in host])
    np.testing.assert_array_equal(got[0], ref[0])
    np.testing.assert_array_equal(got[1], ref[1])
    for k, value, code in ((0, 99.0, VD_ERANGE), (1, np.nan, VD_EINVAL), (2, np.inf, VD_EINVAL),
                           (3, -1.0, VD_EINVAL), (4, -99.0, VD_ERANGE), (5, np.nan, VD_EINVAL)):
        if len(host[k]) == 0:
            continue
        bad = [np.array(x) for x in host]
        bad[k].reshape(-1)[-1] = value
        for arrays in (bad, [shifted(x) for x in bad]):
            with pytest.raises(VDError) as ei:
                solved(arrays)
            assert ei.value.code == code


def _tiles(dims, tile):
    return int(np.prod([-(-n // t) for n, t in zip(dims, tile)]))


@pytest.mark.parametrize("tile", [(8, 8, 4), (16, 4, 8)])
@pytest.mark.parametrize("precision,active", [("fp32", False), ("fp32", True), ("fp64", False),
                                              ("fp64", True)])
def test_abandoned_solves_with_late_workgroups(tile, precision, active):
    """Every second workgroup of an abandoned solve starts only when the tickets
    of the others are 2 to 8 iterates ahead (and at once after the last one):
    the bits of one launch per iteration."""
    dims, pcg = (37, 11, 18), 11
    scene = make_tiny(seed=5, dims=dims, num_levels=1, gn=2, pcg=pcg, n_dense=3000,
                      n_sparse=20, spacing=0.6, origin=(0.2, -1.0, 0.4))
    kw = dict(tiles=({(8, 8, 4): 1, (16, 4, 8): 7}[tile],), precision=precision,
              active_set=active)
    ref = make_lattice(scene, iterative=True, **kw)
    e = ref.solve_frame(reset=True, report=True)["energy"]
    n = _tiles(dims, tile)
    lat = make_lattice(scene, **kw)
    for late in (1, 2 * n, 3 * n, 3 * n + 1, 4 * n, 5 * n + n // 2, 6 * n, 7 * n + 1, 8 * n,
                 (pcg + 1) * n):
        lat.debug_abandon_loops(1 + late)
        rep = lat.solve_frame(reset=True, report=True)
        assert not rep["bits"] & 16
        np.testing.assert_array_equal(rep["energy"], e)
        np.testing.assert_array_equal(lat.get_state64()[0], ref.get_state64()[0])


@pytest.mark.parametrize("active", [False, True])
@pytest.mark.parametrize("dims", [(65, 64, 65), (79, 71, 80)])
def test_abandoned_large_solves_with_late_workgroups(dims, active):
    """The same on tiles of 16x16x8, against the solve that is not abandoned (the
    launches per iteration add the same sums up in another order)."""
    scene = make_tiny(seed=7, dims=dims, num_levels=1, gn=2, pcg=9,
                      n_dense=300 if active else 12000, n_sparse=20,
                      spacing=0.5, origin=(0.2, -1.0, 0.4))
    lat = make_lattice(scene, active_set=active)
    e = lat.solve_frame(reset=True, report=True)["energy"]
    ref = lat.get_state64()[0]
    n = _tiles(dims, (16, 16, 8))
    for late in (2 * n, 3 * n + 1, 4 * n, 6 * n, 8 * n):
        lat.debug_abandon_loops(1 + late)
        rep = lat.solve_frame(reset=True, report=True)
        assert not rep["bits"] & 16
        np.testing.assert_array_equal(rep["energy"], e)
        np.testing.assert_array_equal(lat.get_state64()[0], ref)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("sizes", [(80, 64), (64, 64), (96, 40), (48, 16)])
def test_solves_on_two_streams_equal_solves_alone(sizes, graph):
    """Frames of two lattices whose solves cannot all be resident together, on
    two streams: each has the bits it has alone."""
    import torch
    lats, alone = [], []
    for k, n in enumerate(sizes):
        scene = make_tiny(seed=20 + k, dims=(n, n - 1, n), num_levels=2, gn=3, pcg=25,
                          n_dense=4000, n_sparse=20, spacing=0.5)
        stream = torch.cuda.Stream()
        lat = make_lattice(scene, graph=graph, stream=stream.cuda_stream)
        lat.stream_object = stream
        lat.solve_frame(reset=True)
        torch.cuda.synchronize()
        alone.append(lat.get_state64()[0])
        lats.append(lat)
    for repeat in range(4):
        for frame in range(3):
            for lat in lats if (repeat + frame) % 2 else lats[::-1]:
                lat.solve_frame(reset=True)
        torch.cuda.synchronize()
        for lat, ref in zip(lats, alone):
            np.testing.assert_array_equal(lat.get_state64()[0], ref)


def test_solves_beside_foreign_kernels_equal_solves_alone():
    """A kernel of another stream holds a compute unit for 1.5 to 3.5 ms, so that
    the last workgroup of a solve on all of them (256 tiles, 30 iterations, which
    is abandoned after 1.8 ms) starts while the others are at work on it."""
    import torch
    scene = make_tiny(seed=31, dims=(64, 64, 64), num_levels=1, gn=1, pcg=30, n_dense=4000,
                      n_sparse=20, spacing=0.5)
    lat = make_lattice(scene, tiles=(5,))
    lat.solve_frame(reset=True)
    ref = lat.get_state64()[0]
    side = torch.cuda.Stream()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with torch.cuda.stream(side):
        torch.cuda._sleep(1000)
        a.record()
        torch.cuda._sleep(1_000_000)
        b.record()
    side.synchronize()
    per_ms = 1_000_000 / a.elapsed_time(b)
    for ms in np.linspace(1.5, 3.5, 41):
        with torch.cuda.stream(side):
            torch.cuda._sleep(int(ms * per_ms))
        rep = lat.solve_frame(reset=True, report=True)
        torch.cuda.synchronize()
        assert not rep["bits"] & 16
        np.testing.assert_array_equal(lat.get_state64()[0], ref)


def test_solves_of_many_iterations_on_two_streams_equal_launches_per_iteration():
    """Solves of 64^3 that take longer than a millisecond each, on two streams and
    in both precisions: the bits of one launch per iteration."""
    import torch
    lats, refs = [], []
    for k, precision in enumerate(("fp32", "fp64", "fp32")):
        scene = make_tiny(seed=40 + k, dims=(64, 63, 64), num_levels=1, gn=2, pcg=120,
                          n_dense=4000, n_sparse=20, spacing=0.5)
        ref = make_lattice(scene, precision=precision, tiles=(6,), iterative=True)
        ref.solve_frame(reset=True)
        refs.append(ref.get_state64()[0])
        lats.append(make_lattice(scene, precision=precision, tiles=(6,),
                                 stream=torch.cuda.Stream().cuda_stream))
    torch.cuda.synchronize()
    for lat in lats * 3:
        lat.solve_frame(reset=True)
    torch.cuda.synchronize()
    for lat, ref in zip(lats, refs):
        np.testing.assert_array_equal(lat.get_state64()[0], ref)


@pytest.mark.parametrize("tile", [4, 6, 7, 8])
def test_one_launch_solves_of_tiles_full_of_data_nodes(tile):
    """A lattice whose every node carries data blocks (20-40 tiles): the bits of
    one launch per iteration."""
    scene = make_tiny(seed=13, dims=(24, 20, 16), num_levels=1, gn=2, pcg=8, n_dense=20000,
                      n_sparse=40, spacing=0.5, origin=(0.3, 0.1, -0.2))
    out = {}
    for iterative in (True, False):
        lat = make_lattice(scene, tiles=(tile,), iterative=iterative)
        rep = lat.solve_frame(report=True)
        assert not rep["bits"] & 16
        out[iterative] = (rep["energy"], lat.get_state64()[0])
    np.testing.assert_array_equal(out[False][0], out[True][0])
    np.testing.assert_array_equal(out[False][1], out[True][1])
