"""GPU checks of the batched entry points: many submaps and robots per launch.

The batched path runs the same per-element arithmetic as the single-map
path, so its outputs must be identical bit for bit; selected items are also
checked against the oracle.  Graph replays must reproduce the eager result."""
import sys

import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[gpu] {msg}", file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_07631_amd as P
    P.lib()
    return P


def bits(t):
    a = t.detach().cpu().numpy()
    return a.view(np.uint32) if a.dtype == np.float32 else a


def make_batch(seed, n_items, side_hi=160, pts_hi=120_000, extra_empty=True):
    items = scenes.submap_batch(seed, n_items, side_lo=20, side_hi=side_hi, pts_lo=2_000, pts_hi=pts_hi)
    if extra_empty:
        # an item whose points all lie outside its grid, and an item with no points
        junk = scenes.Scene(np.array([[-50.0, -50.0, 1.0]], np.float32),
                            dict(x0=0.0, y0=0.0, res=0.1, nx=30, ny=20, slice_dz=0.3))
        none = scenes.Scene(np.zeros((0, 3), np.float32), dict(x0=0.0, y0=0.0, res=0.1, nx=7, ny=9, slice_dz=0.3))
        items = items[:2] + [junk] + items[2:] + [none]
    pts, specs, off = [], [], 0
    for sc in items:
        specs.append(dict(xyz_offset=off, n_points=len(sc.points), grid=sc.grid))
        pts.append(sc.points)
        off += len(sc.points)
    return items, np.ascontiguousarray(np.concatenate(pts)), specs


def test_batched_equals_single(P, oracle_lib):
    import torch
    items, pts, specs = make_batch(61, 14)
    xyz = torch.from_numpy(pts).cuda()
    rb = P.robot_from_physical(scenes.ROBOT_CONFIG0, 0.1)
    say(f"batch of {len(specs)} submaps, {len(pts)} points")
    b = P.Batch(xyz, specs, n_robots=1, with_ids=True)
    P.pct_tomogram_extent_batched(b)
    G, Cc, aG, aC = P.pct_build_tomogram_batched(b, with_ids=True)
    cost, keep = P.pct_eval_traversability_batched(b, G, Cc, [rb])
    torch.cuda.synchronize()
    for i, (sc, sp) in enumerate(zip(items, specs)):
        sub = xyz[sp["xyz_offset"]:sp["xyz_offset"] + sp["n_points"]]
        ext = P.pct_tomogram_extent(sub, sp["grid"]) if sp["n_points"] else P.pct_extent(0, 0, 0, 0, 0, 0)
        it = b.items[i]
        assert it.extent.n_slices == ext.n_slices and it.extent.n_used == ext.n_used
        if ext.n_slices == 0:
            continue
        assert it.extent.z_min == ext.z_min and it.extent.z_max == ext.z_max
        g1, c1, a1, a2 = P.pct_build_tomogram(sub, sp["grid"], ext, with_ids=True)
        np.testing.assert_array_equal(bits(b.item_view(G, i)), bits(g1))
        np.testing.assert_array_equal(bits(b.item_view(Cc, i)), bits(c1))
        # batched ids index the shared point array
        np.testing.assert_array_equal(bits(b.item_view(aG, i)), np.where(bits(a1) >= 0, bits(a1) + sp["xyz_offset"], -1))
        np.testing.assert_array_equal(bits(b.item_view(aC, i)), np.where(bits(a2) >= 0, bits(a2) + sp["xyz_offset"], -1))
        cs, ks = P.pct_eval_traversability(g1, c1, sp["grid"], ext, [rb])
        np.testing.assert_array_equal(bits(b.item_view(cost[0], i)), bits(cs[0]))
        ko = it.keep_offset
        np.testing.assert_array_equal(bits(keep[0, ko:ko + ext.n_slices]), bits(ks[0]))
        if i < 3:
            tm = oracle_lib.tomogram(sc.points, sp["grid"])
            np.testing.assert_array_equal(bits(g1), tm["ground"].view(np.uint32))



@pytest.mark.parametrize("ids", [True, False])
def test_batched_scatter_edges(P, oracle_lib, ids):
    """Items of one tile, of exactly and one more than the most tiles whose
    scatter is staged in LDS (1024), chunks of 4095 to 4097 points, and every
    alignment of an item's points, against the oracle."""
    import torch
    rng = np.random.default_rng(8)
    shapes = [(64, 8, 4095), (300, 1024, 4097), (300, 1026, 9001), (129, 3, 1), (1, 1, 4096), (256, 4, 2), (50, 60, 4099)]
    specs, pts, off = [], [], 0
    for nx, ny, n in shapes:
        p = np.stack([rng.uniform(-0.05, 0.1 * nx + 0.05, n), rng.uniform(-0.05, 0.1 * ny + 0.05, n),
                      rng.uniform(0.0, 2.5, n)], 1).astype(np.float32)
        specs.append(dict(xyz_offset=off, n_points=n, grid=dict(x0=0.0, y0=0.0, res=0.1, nx=nx, ny=ny, slice_dz=0.3)))
        pts.append(p)
        off += n
    b = P.Batch(torch.from_numpy(np.concatenate(pts)).cuda(), specs, n_robots=1, with_ids=ids)
    P.pct_tomogram_extent_batched(b)
    G, Cc, aG, aC = P.pct_build_tomogram_batched(b, with_ids=ids)
    for i, (p, sp) in enumerate(zip(pts, specs)):
        tm = oracle_lib.tomogram(p, sp["grid"])
        assert b.items[i].extent.n_slices == len(tm["h"])
        if not len(tm["h"]):
            continue
        np.testing.assert_array_equal(bits(b.item_view(G, i)), tm["ground"].view(np.uint32))
        np.testing.assert_array_equal(bits(b.item_view(Cc, i)), tm["ceil"].view(np.uint32))
        if ids:
            for got, want in ((aG, tm["arg_ground"]), (aC, tm["arg_ceil"])):
                np.testing.assert_array_equal(bits(b.item_view(got, i)), np.where(want >= 0, want + sp["xyz_offset"], -1))


def test_batched_many_robots(P):
    """One map, several robot profiles in one launch = one call per robot."""
    import torch
    sc = scenes.multistorey_scene(62, 11.7, 8.3, 700_000, n_floors=3)
    xyz = torch.from_numpy(sc.points).cuda()
    profiles = scenes.robot_profiles(4, 6)
    rbs = [P.robot_from_physical(p, 0.1) for p in profiles]
    say("batched robot profiles")
    b = P.Batch(xyz, [dict(xyz_offset=0, n_points=len(sc.points), grid=sc.grid)], n_robots=len(rbs))
    P.pct_tomogram_extent_batched(b)
    G, Cc, _, _ = P.pct_build_tomogram_batched(b)
    cost, keep = P.pct_eval_traversability_batched(b, G, Cc, rbs)
    ext = b.items[0].extent
    g1 = b.item_view(G, 0).contiguous()
    c1 = b.item_view(Cc, 0).contiguous()
    for r, rb in enumerate(rbs):
        cs, ks = P.pct_eval_traversability(g1, c1, sc.grid, ext, [rb])
        np.testing.assert_array_equal(bits(b.item_view(cost[r], 0)), bits(cs[0]))
        np.testing.assert_array_equal(bits(keep[r, :ext.n_slices]), bits(ks[0]))


@pytest.mark.parametrize("res", [(0.1, 0.2, 0.1, 0.1), (0.2, 0.2, 0.1, 0.25)])
def test_batched_resolutions(P, res):
    """Items of several resolutions and an item without points between them,
    two robots: every item takes its own resolution's weights."""
    import torch
    rng = np.random.default_rng(19)
    specs, pts, off = [], [], 0
    for i, r in enumerate(res):
        n = 0 if i == 2 else 9000
        p = (rng.uniform(0.0, 1.0, (n, 3)) * [70 * r, 50 * r, 2.5]).astype(np.float32)
        specs.append(dict(xyz_offset=off, n_points=n, grid=dict(x0=0.0, y0=0.0, res=r, nx=70, ny=50, slice_dz=0.3)))
        pts.append(p)
        off += n
    rbs = [P.robot_from_physical(p, 0.1) for p in scenes.robot_profiles(5, 2)]
    b = P.Batch(torch.from_numpy(np.concatenate(pts)).cuda(), specs, n_robots=2)
    P.pct_tomogram_extent_batched(b)
    G, Cc, _, _ = P.pct_build_tomogram_batched(b)
    cost, keep = P.pct_eval_traversability_batched(b, G, Cc, rbs)
    for i, sp in enumerate(specs):
        ext = b.items[i].extent
        if ext.n_slices == 0:
            continue
        for r, rb in enumerate(rbs):
            cs, _ = P.pct_eval_traversability(b.item_view(G, i).contiguous(), b.item_view(Cc, i).contiguous(),
                                              sp["grid"], ext, [rb])
            np.testing.assert_array_equal(bits(b.item_view(cost[r], i)), bits(cs[0]))


def test_graph_capture_replays(P):
    """The batched build and evaluation captured in one graph; every replay,
    with eager work and synchronisation in between, equals the eager run."""
    import torch
    items, pts, specs = make_batch(63, 8, extra_empty=False)
    xyz = torch.from_numpy(pts).cuda()
    rb = P.robot_from_physical(scenes.ROBOT_CONFIG0, 0.1)
    b = P.Batch(xyz, specs)
    P.pct_tomogram_extent_batched(b)
    G, Cc, _, _ = P.pct_build_tomogram_batched(b)
    cost, keep = P.pct_eval_traversability_batched(b, G, Cc, [rb])
    torch.cuda.synchronize()
    ref = [t.clone() for t in (G, Cc, cost, keep)]
    outs = (torch.empty_like(G), torch.empty_like(Cc), None, None)
    couts = (torch.empty_like(cost), torch.empty_like(keep))
    say("graph capture")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        # warm-up on the capture stream, then capture with resident descriptors
        P.pct_build_tomogram_batched(b, out=outs)
        P.pct_eval_traversability_batched(b, outs[0], outs[1], [rb], out=couts)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            P.pct_build_tomogram_batched(b, flags=P.PCT_DESCRIPTORS_RESIDENT, out=outs)
            P.pct_eval_traversability_batched(b, outs[0], outs[1], [rb], flags=P.PCT_DESCRIPTORS_RESIDENT, out=couts)
    for rep in range(3):
        for t in (*outs[:2], *couts):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, r in zip((*outs[:2], *couts), ref):
            assert torch.equal(a.view(torch.uint8), r.view(torch.uint8)), f"replay {rep} differs"
        _ = (xyz * 2.0).sum().item()      # unrelated eager work between replays


def test_batch_tuning_changes_no_output(P, tmp_path):
    """The size-class tuner records one tile height and one strip shape per
    class; the batched outputs (with ids and slice flags) after tuning, after
    loading other shapes from a file and in a graph captured with the tuned
    shapes are those before tuning, bit for bit; descriptor tables uploaded
    with other shapes are refused for resident calls."""
    import torch
    items, pts, specs = make_batch(65, 24, side_hi=300, pts_hi=150_000)
    xyz = torch.from_numpy(pts).cuda()
    rb = P.robot_from_physical(scenes.ROBOT_CONFIG0, 0.1)
    P.pct_autotune_reset()
    b = P.Batch(xyz, specs, n_robots=1, with_ids=True)
    P.pct_tomogram_extent_batched(b)

    def run(flags=0, out=None):
        G, Cc, aG, aC = P.pct_build_tomogram_batched(b, with_ids=True, flags=flags, out=out and out[:4])
        cost, keep = P.pct_eval_traversability_batched(b, G, Cc, [rb], flags=flags, out=out and out[4:])
        return [G, Cc, aG, aC, cost, keep]

    ref = [t.clone() for t in run()]
    torch.cuda.synchronize()
    say(f"tuning a batch of {len(specs)} submaps")
    ent = P.pct_autotune_batched(b, rb)
    classes = {(e["stage"], e["class_x"], e["class_y"], e["radius"]) for e in ent}
    assert {c[0] for c in classes} == {"build", "eval"} and len(classes) >= 4
    chosen = {}
    for c in classes:
        ch = [e for e in ent if (e["stage"], e["class_x"], e["class_y"], e["radius"]) == c and e["chosen"]]
        assert len(ch) == 1, c
        chosen[c] = (ch[0]["rows"], ch[0]["waves"])
    say(f"{len(ent)} timings over {len(classes)} (stage, class) pairs")

    def same(outs, what):
        torch.cuda.synchronize()
        for a, r in zip(outs, ref):
            assert torch.equal(a.view(torch.uint8), r.view(torch.uint8)), what

    same(run(), "after tuning")
    # other shapes for every class, from a file
    it0 = next(it for it in b.items if it.extent.n_slices > 0)
    P.pct_autotune_set_traversability(it0.grid, it0.extent, rb, 64, 1)   # at least one record
    tuned = tmp_path / "tuned.txt"
    P.pct_autotune_save(tuned)
    recs = [l.split() for l in tuned.read_text().splitlines() if l and not l.startswith("#")]
    assert recs, "the tuner recorded nothing"
    arch = recs[0][0]       # the device's architecture tag
    lines = []
    for (st, cx, cy, R), ch in sorted(chosen.items()):
        if st == "build":
            lines.append(f"{arch} batch_build {cx} {cy} {4 if ch[0] == 8 else 8}")
        else:
            lines.append(f"{arch} batch_eval {cx} {cy} {R} {64 if ch == (32, 1) else 32} 1")
    path = tmp_path / "tune.txt"
    path.write_text("\n".join(lines) + "\n")
    assert P.pct_autotune_load(path) == len(lines)
    with pytest.raises(P.PctError):
        run(P.PCT_DESCRIPTORS_RESIDENT, [torch.empty_like(t) for t in ref])
    same(run(), "with loaded shapes")
    # a graph captured with these shapes
    outs = [torch.empty_like(t) for t in ref]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        run(0, outs)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            run(P.PCT_DESCRIPTORS_RESIDENT, outs)
    for rep in range(2):
        for t in outs:
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        same(outs, f"graph replay {rep}")
    # save and load back
    saved = tmp_path / "saved.txt"
    P.pct_autotune_save(saved)
    n_rec = len([l for l in saved.read_text().splitlines() if l and not l.startswith("#")])
    assert n_rec >= len(lines) + 1
    P.pct_autotune_reset()
    assert P.pct_autotune_load(saved) == n_rec
    P.pct_autotune_reset()


def test_graph_capture_with_library_helpers(P):
    """The same capture through the C ABI's pct_graph_begin / pct_graph_end:
    every replay equals the eager run; an empty capture replays as a no-op."""
    import torch
    items, pts, specs = make_batch(64, 6, extra_empty=False)
    xyz = torch.from_numpy(pts).cuda()
    rb = P.robot_from_physical(scenes.ROBOT_CONFIG0, 0.1)
    b = P.Batch(xyz, specs)
    P.pct_tomogram_extent_batched(b)
    G, Cc, _, _ = P.pct_build_tomogram_batched(b)
    cost, keep = P.pct_eval_traversability_batched(b, G, Cc, [rb])
    torch.cuda.synchronize()
    ref = [t.clone() for t in (G, Cc, cost, keep)]
    outs = (torch.empty_like(G), torch.empty_like(Cc), None, None)
    couts = (torch.empty_like(cost), torch.empty_like(keep))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        P.pct_build_tomogram_batched(b, out=outs)
        P.pct_eval_traversability_batched(b, outs[0], outs[1], [rb], out=couts)
        torch.cuda.synchronize()
        graph = P.Graph(s)
        with graph:
            P.pct_build_tomogram_batched(b, flags=P.PCT_DESCRIPTORS_RESIDENT, out=outs)
            P.pct_eval_traversability_batched(b, outs[0], outs[1], [rb], flags=P.PCT_DESCRIPTORS_RESIDENT, out=couts)
        empty = P.Graph(s)
        with empty:
            pass
    for rep in range(3):
        for t in (*outs[:2], *couts):
            t.zero_()
        torch.cuda.synchronize()
        graph.launch(s)
        empty.launch(s)
        s.synchronize()
        for a, r in zip((*outs[:2], *couts), ref):
            assert torch.equal(a.view(torch.uint8), r.view(torch.uint8)), f"replay {rep} differs"
        _ = (xyz * 2.0).sum().item()      # unrelated eager work between replays
    del graph, empty


def test_full_size_submap_batch(P, oracle_lib):
    """512 submaps of 50-400 cells and 10k-1M points (the batching
    workload), batched in the benchmark's configuration; every 32nd item is
    compared with the single-map path and three with the oracle."""
    import torch
    items = scenes.submap_batch(3, 512)
    pts, specs, off = [], [], 0
    for sc in items:
        specs.append(dict(xyz_offset=off, n_points=len(sc.points), grid=sc.grid))
        pts.append(sc.points)
        off += len(sc.points)
    xyz = torch.from_numpy(np.ascontiguousarray(np.concatenate(pts))).cuda()
    rb = P.robot_from_physical(scenes.ROBOT_CONFIG0, 0.1)
    say(f"full-size submap batch: {len(specs)} items, {off} points")
    b = P.Batch(xyz, specs)
    P.pct_tomogram_extent_batched(b)
    G, Cc, _, _ = P.pct_build_tomogram_batched(b)
    cost, keep = P.pct_eval_traversability_batched(b, G, Cc, [rb])
    torch.cuda.synchronize()
    for i in range(0, 512, 32):
        sp = specs[i]
        sub = xyz[sp["xyz_offset"]:sp["xyz_offset"] + sp["n_points"]]
        ext = P.pct_tomogram_extent(sub, sp["grid"])
        g1, c1, _, _ = P.pct_build_tomogram(sub, sp["grid"], ext)
        np.testing.assert_array_equal(bits(b.item_view(G, i)), bits(g1))
        cs, ks = P.pct_eval_traversability(g1, c1, sp["grid"], ext, [rb])
        np.testing.assert_array_equal(bits(b.item_view(cost[0], i)), bits(cs[0]))
        if i in (0, 256, 480):
            tm = oracle_lib.tomogram(items[i].points, sp["grid"])
            np.testing.assert_array_equal(bits(g1), tm["ground"].view(np.uint32))
            lo, hi, _ = oracle_lib.envelope(tm["ground"], tm["ceil"], 0.1, rb.as_dict())
            c = cs[0].cpu().numpy().astype(np.float64)
            assert np.all(c >= lo - 1e-5) and np.all(c <= hi + 1e-5)


@pytest.mark.parametrize("ids", [True, False])
def test_batched_scatter_of_many_tiles(P, oracle_lib, ids):
    """Items of more tiles than a staged scatter takes, up to the most whose
    tiles are counted in LDS (8192) and beyond, beside a small one."""
    import torch
    rng = np.random.default_rng(9)
    shapes = [(300, 1026, 4096), (129, 16384, 9001), (300, 33000, 12289), (40, 30, 700)]   # 1026, 8192, 8250, 4 tiles
    specs, pts, off = [], [], 0
    for nx, ny, n in shapes:
        p = np.stack([rng.uniform(-0.05, 0.1 * nx + 0.05, n), rng.uniform(-0.05, 0.1 * ny + 0.05, n),
                      rng.uniform(0.0, 0.5, n)], 1).astype(np.float32)
        p[: n // 2, 1] = rng.uniform(0.0, 0.4, n // 2)       # many records in few tiles as well
        specs.append(dict(xyz_offset=off, n_points=n, grid=dict(x0=0.0, y0=0.0, res=0.1, nx=nx, ny=ny, slice_dz=0.3)))
        pts.append(p)
        off += n
    b = P.Batch(torch.from_numpy(np.concatenate(pts)).cuda(), specs, n_robots=1, with_ids=ids)
    P.pct_tomogram_extent_batched(b)
    G, Cc, aG, aC = P.pct_build_tomogram_batched(b, with_ids=ids)
    for i, (p, sp) in enumerate(zip(pts, specs)):
        tm = oracle_lib.tomogram(p, sp["grid"])
        assert b.items[i].extent.n_slices == len(tm["h"])
        np.testing.assert_array_equal(bits(b.item_view(G, i)), tm["ground"].view(np.uint32))
        np.testing.assert_array_equal(bits(b.item_view(Cc, i)), tm["ceil"].view(np.uint32))
        if ids:
            for got, want in ((aG, tm["arg_ground"]), (aC, tm["arg_ceil"])):
                np.testing.assert_array_equal(bits(b.item_view(got, i)), np.where(want >= 0, want + sp["xyz_offset"], -1))


@pytest.mark.parametrize("R", range(0, 9))
def test_default_strips_change_no_cost(P, R):
    """The default strips of a map (one, two or four wavefronts, by radius and
    size) and of a batch (one wavefront, or four on wide maps) give the costs
    of explicit shapes, bit for bit, and the same kept slices."""
    import torch
    rng = np.random.default_rng(R)
    inf = {0: (0.0, 0.15), 1: (0.0, 0.25), 2: (0.0, 0.4)}.get(R, (0.05 + 0.1 * (R - 3), 0.4))
    r = dict(d_min=0.5, d_ref=0.65, theta_b=1.7, theta_s=0.36, theta_p=0.2, c_barrier=50.0, alpha_d=20.0, alpha_b=20.0,
             alpha_s=15.0, d_inf=inf[0], d_sm=inf[1], patch_radius=1)
    assert P.pct_kernel_radius(r, 0.1) == R
    shapes = [(512, 33), (700, 431), (1500, 90), (45, 300), (511, 20)]
    pts, specs, off = [], [], 0
    for nx, ny in shapes:
        n = 3 * nx * ny
        z = 3.0 * rng.integers(0, 3, n) + rng.normal(0.0, 0.02, n)
        p = np.stack([rng.uniform(0.0, 0.1 * nx, n), rng.uniform(0.0, 0.1 * ny, n), z], 1).astype(np.float32)
        specs.append(dict(xyz_offset=off, n_points=n, grid=dict(x0=0.0, y0=0.0, res=0.1, nx=nx, ny=ny, slice_dz=0.3)))
        pts.append(p)
        off += n
    b = P.Batch(torch.from_numpy(np.concatenate(pts)).cuda(), specs, n_robots=1)
    P.pct_tomogram_extent_batched(b)
    G, Cc, _, _ = P.pct_build_tomogram_batched(b)
    cost, keep = P.pct_eval_traversability_batched(b, G, Cc, [r])
    for i, sp in enumerate(specs):
        ext, g = b.items[i].extent, sp["grid"]
        gi, ci = b.item_view(G, i).contiguous(), b.item_view(Cc, i).contiguous()
        want, kept = P.pct_eval_traversability(gi, ci, g, ext, [r])
        assert torch.equal(b.item_view(cost[0], i).view(torch.int32), want[0].view(torch.int32)), (g["nx"], g["ny"])
        ko = b.items[i].keep_offset
        assert torch.equal(keep[0][ko:ko + ext.n_slices], kept[0]), (g["nx"], g["ny"])
        for rows, waves in ((256, 4), (64, 2), (16, 1)):
            P.pct_autotune_set_traversability(g, ext, r, rows, waves)
            other, kept2 = P.pct_eval_traversability(gi, ci, g, ext, [r])
            assert torch.equal(other.view(torch.int32), want.view(torch.int32)) and torch.equal(kept2, kept), (rows, waves)
        P.pct_autotune_reset()
