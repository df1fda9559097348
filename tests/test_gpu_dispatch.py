"""GPU parity with the oracle on the sizes where a kernel changes its way of
working: hand-made frames of many separate charts, each at the edge of a rule."""
import numpy as np
import pytest
import torch

import oracle
from synth import scenes
from test_gpu_parity import _fa, compare

pytestmark = pytest.mark.gpu


def fans(owners, seed=0, atlas_size=1024, side=1.6, width=1280, height=720):
    """A frame of flat triangle fans facing the camera: triangle i belongs to fan
    owners[i] (fans share no vertex, triangles of a fan share its centre), laid
    out on a square grid of `side` over the view."""
    owners = np.asarray(owners)
    n = int(owners.max()) + 1
    k = int(np.ceil(np.sqrt(n)))
    rng = np.random.default_rng(seed)
    cell = side / k
    cx = (np.arange(n) % k + 0.5) * cell - side / 2
    cy = (np.arange(n) // k + 0.5) * cell - side / 2
    count = np.bincount(owners, minlength=n)
    first = np.concatenate([[0], np.cumsum(count + 2)])  # centre, then count + 1 rim vertices
    pos = np.zeros((first[-1], 3))
    tris = np.zeros((len(owners), 3), np.int64)
    for c in range(n):
        ang = np.linspace(0, min(1.9 * np.pi, 1.2 * count[c]), count[c] + 1)
        rad = cell * rng.uniform(0.2, 0.48) * rng.uniform(0.7, 1.0, count[c] + 1)
        b = first[c]
        pos[b, :2] = cx[c], cy[c]
        pos[b + 1:b + 2 + count[c], 0] = cx[c] + rad * np.cos(ang)
        pos[b + 1:b + 2 + count[c], 1] = cy[c] + rad * np.sin(ang)
    at = np.zeros(n, np.int64)
    for i, c in enumerate(owners):
        tris[i] = first[c], first[c] + 1 + at[c], first[c] + 2 + at[c]
        at[c] += 1
    cam = scenes.make_camera((0.0, 0.0, 2.0), (0.0, 0.0, 0.0), width, height, 0.05, 100.0, up=(0, 1, 0))
    pos, tris = pos.astype(np.float32), tris.astype(np.int32)
    vis = scenes.visible_set(pos, tris, cam)
    assert vis.all()
    return scenes.Frame(f"fans{n}/{len(owners)}", pos, tris, vis, cam.view_proj, width, height,
                        atlas_size, 1.0, 991, cam.eye, cam.near, 0)


def check(frame, J=64, gutter=1, flags=0, min_box=2, **context):
    fa = _fa()
    print(f"[gpu] {frame.name} omega={frame.atlas_size} J={J} flags={flags} {context}", flush=True)
    ctx = fa.Context(frame.num_triangles, frame.num_vertices, max_charts=65536, max_atlas=8192,
                     num_scales=J, gutter=gutter, flags=flags, min_box=min_box, tuning_table=None,
                     **context)
    mesh = fa.Mesh(frame.positions, frame.indices, frame.scene_key)
    out = ctx.build_atlas(mesh, torch.as_tensor(frame.visible).cuda(), frame.view_proj,
                          frame.width, frame.height, frame.atlas_size, frame.rate)
    torch.cuda.synchronize()
    g = out.to_numpy()
    ctx.close()
    return g


# the box gather reduces a chart in registers from 8 lanes of a wave up
@pytest.mark.parametrize("per", [1, 7, 8, 9, 63, 64, 65])
def test_gather_group_sizes(per):
    f = fans(np.repeat(np.arange(1300 // per + 1), per), seed=per)
    compare(check(f), oracle.build_frame(f))


def test_gather_table_overflow():
    # one workgroup (list entries 1024..2047) names charts 1024..1535 and
    # 0..511: two charts for each of 512 neighbouring table slots, so the
    # second ones run out of probes and go to the global words
    f = fans(np.concatenate([np.arange(1536), np.arange(512)]), atlas_size=2048)
    compare(check(f), oracle.build_frame(f))


# the occupied texels are counted per strip of 64 atlas columns, up to the
# strip's highest box: maps narrower than a strip, of one row of words per
# workgroup (4096) and of two (8192)
@pytest.mark.parametrize("omega,n", [(16, 3), (32, 7), (64, 20), (128, 5), (4096, 30), (8192, 300)])
def test_occupied_texels(omega, n):
    f = fans(np.repeat(np.arange(n), 3), seed=omega, atlas_size=omega)
    g = check(f)
    assert g["meta"]["status"] == 0
    assert g["meta"]["occupied_texels"] == int((g["occupancy"] >= 0).sum()) > 0
    compare(g, oracle.build_frame(f))


# Triangles whose vertices are within 512 texels of the first one are tested in
# 32 bits, larger ones in 64: fans of a few triangles whose sides go from
# beyond 2000 texels to below 60, some of them on both sides of 512.
@pytest.mark.parametrize("n,per", [(1, 1), (1, 2), (1, 5), (2, 3), (4, 5), (5, 1), (9, 4), (12, 5),
                                   (16, 3), (25, 5), (36, 2), (400, 5)])
@pytest.mark.parametrize("omega", [2048, 8192])
def test_occupancy_sides(n, per, omega):
    f = fans(np.arange(n * per) // per, seed=n + per, atlas_size=omega, width=3840, height=2160)
    compare(check(f), oracle.build_frame(f))


# Footprints drawn by the whole wave, 64 texels at a time, likewise: all of them
# up to 4096 texels, within 512 texels of their first vertex or beyond.
@pytest.mark.parametrize("n,per", [(1, 1), (4, 5), (9, 4), (36, 2), (400, 5), (3000, 1)])
@pytest.mark.parametrize("omega", [256, 2048, 8192])
def test_occupancy_expanded(n, per, omega):
    fa = _fa()
    f = fans(np.arange(n * per) // per, seed=n + per, atlas_size=omega, width=3840, height=2160)
    print(f"[gpu] expanded {f.name} omega={omega}", flush=True)
    ctx = fa.Context(f.num_triangles, f.num_vertices, max_charts=65536, max_atlas=8192,
                     tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_OCC_LANE_TEXELS, 0)
    ctx.set_tuning(fa.FA_TUNE_OCC_SMALL_TEXELS, 4096)
    out = ctx.build_atlas(fa.Mesh(f.positions, f.indices, f.scene_key),
                          torch.as_tensor(f.visible).cuda(), f.view_proj, f.width, f.height, omega,
                          f.rate)
    torch.cuda.synchronize()
    g = out.to_numpy()
    ctx.close()
    compare(g, oracle.build_frame(f))


# Footprint push: profiles from entries of one triangle to whole groups of 64,
# of charts from a few columns to more than a window, charts over and under the
# width that a whole workgroup pushes, gutters of 1 to 5, and lists longer than
# the records' memory (more than 2^20 entries are set up again).
@pytest.mark.parametrize("owners,omega,gutter", [
    (np.arange(1), 256, 1), (np.arange(63), 512, 1), (np.arange(200) // 3, 1024, 1),
    (np.arange(6) // 3, 4096, 2), (np.arange(3), 8192, 5), (np.arange(40) // 5, 8192, 3),
    (np.arange(5000) // 2, 4096, 1)])
def test_footprint_sizes(owners, omega, gutter):
    f = fans(owners, seed=len(owners), atlas_size=omega, width=3840, height=2160)
    g = check(f, gutter=gutter, flags=4)
    compare(g, oracle.build_frame(f, gutter=gutter, footprint=True))


def test_footprint_long_list():
    n = 730
    y, x = np.mgrid[0:n + 1, 0:n + 1] / n * 2 - 1
    pos = np.stack([x, y, 0.1 * np.sin(5 * x) * np.cos(4 * y)], -1).reshape(-1, 3)
    v = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).reshape(-1)
    tris = np.stack([v, v + 1, v + n + 2, v, v + n + 2, v + n + 1], 1).reshape(-1, 3)
    assert len(tris) > 1 << 20
    cam = scenes.make_camera((0.0, 0.0, 2.5), (0.0, 0.0, 0.0), 1920, 1080, 0.05, 100.0,
                             up=(0, 1, 0))
    f = scenes.Frame("long list", pos.astype(np.float32), tris.astype(np.int32),
                     np.ones(len(tris), np.uint8), cam.view_proj, 1920, 1080, 1024, 1.0, 992,
                     cam.eye, cam.near, 0)
    compare(check(f, flags=4), oracle.build_frame(f, footprint=True))


# The box push goes by rows (each box rests on the few boxes of the row before)
# or by columns (a whole frontline): by columns up to 8 boxes, with overflows
# above 1024 columns and where two rows may not fit a chunk. Other edges: chunks
# of 8128 boxes (and stop checks at multiples of another number), boxes over
# more than 8 and 16 others, more than 8 boxes of a row over edge columns.
def _uniform(n, lo, hi, seed=0):
    return np.random.default_rng(seed).uniform(lo, hi, (n, 2))


def _thin_and_square(seed=1):
    rng = np.random.default_rng(seed)
    thin = np.stack([rng.uniform(1, 3, 900), rng.uniform(99, 101, 900)], 1)
    return rng.permutation(np.concatenate([thin, rng.uniform(60, 98, (200, 2))]))


def _narrow_and_wide(n, side, seed=2):
    # small boxes with a few as wide as `side` among the lowest rows: wide edges
    rng = np.random.default_rng(seed)
    wide = np.stack([rng.uniform(0.5 * side, side, 12), rng.uniform(side, 1.01 * side, 12)], 1)
    return np.concatenate([rng.uniform(1, 9, (n, 2)), wide])


PUSH_CASES = {
    "7 boxes": (_uniform(7, 5, 60), 128, {}),
    "8 boxes": (_uniform(8, 5, 60), 128, {}),
    "9 boxes": (_uniform(9, 5, 60), 128, {}),
    "65 boxes": (_uniform(65, 5, 60), 512, {}),
    "wide overflow": (_uniform(40, 100, 3900), 4096, {}),
    "overflow on both sides of 1024": (_uniform(60, 100, 1400), 4096, {}),
    "rows longer than a chunk": (_uniform(30000, 0.2, 6), 8192, dict(g=0, mmin=1)),
    "rows of a third of a chunk": (_uniform(20000, 0.2, 6), 4096, dict(g=0, mmin=2)),
    "255 boxes": (_uniform(255, 5, 30).round(), 1024, {}),
    "256 boxes": (_uniform(256, 5, 30).round(), 1024, {}),
    "257 boxes": (_uniform(257, 5, 30).round(), 1024, {}),
    "2047 boxes": (_uniform(2047, 1, 30), 2048, {}),
    "2048 boxes": (_uniform(2048, 1, 30), 2048, {}),
    "2049 boxes": (_uniform(2049, 1, 30), 2048, {}),
    "8127 boxes": (_uniform(8127, 1, 30), 4096, {}),
    "8128 boxes": (_uniform(8128, 1, 30), 4096, {}),
    "8129 boxes": (_uniform(8129, 1, 30), 4096, {}),
    "three chunks": (_uniform(24000, 1, 40), 4096, {}),
    "chunks short of the stop checks": (_uniform(22000, 1, 12), 1024, {}),
    "thin under square": (_thin_and_square(), 1024, {}),
    "narrow over wide edges": (_narrow_and_wide(3000, 400), 1024, {}),
    "narrow over very wide edges": (_narrow_and_wide(3000, 900), 2048, {}),
    "tiny atlas": (_uniform(300, 0.5, 4), 16, dict(J=7)),
}


@pytest.mark.parametrize("name", list(PUSH_CASES))
@pytest.mark.parametrize("block", [256, 512, 1024])
def test_push_paths(name, block):
    from test_gpu_parity import _oracle_pack
    fa = _fa()
    sizes, omega, opt = PUSH_CASES[name]
    sizes = sizes.astype(np.float32)
    J, g, mmin = opt.get("J", 64), opt.get("g", 1), opt.get("mmin", 2)
    print(f"[gpu] push {name} n={len(sizes)} omega={omega} block={block}", flush=True)
    ctx = fa.Context(1, 1, max_charts=65536, max_atlas=8192, num_scales=J, gutter=g, min_box=mmin,
                     tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_PACK_BLOCK, block)
    pl, meta, cand = ctx.pack_boxes(torch.as_tensor(sizes).cuda(), omega)
    torch.cuda.synchronize()
    m, c = fa.parse_meta(meta), cand.cpu().numpy()
    pl = pl.cpu().numpy()
    ctx.close()
    js, table, want = _oracle_pack(sizes, omega, J, g, mmin)
    assert m["chosen_j"] == js
    assert np.array_equal(c[:, :3], table[:, :3])
    fit = table[:, 0] == 1
    assert np.array_equal(c[fit, 3], table[fit, 3])
    assert ((c[~fit, 3] == -1) | (c[~fit, 3] > c[~fit, 2])).all()
    if js:
        assert np.array_equal(pl, want)


# Prologue and compaction take four triangles or vertices a lane, a tile of 1024
# triangles a wave and four a workgroup, in wide words where a buffer's address
# allows: sizes around those, hidden triangles in between, and buffers that are
# not aligned to more than their elements.
@pytest.mark.parametrize("T", [8193, 9217, 12287, 12289, 16384, 20002])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_prologue_tiles(T, shift):
    fa = _fa()
    frame = fans(np.arange(T) // 4, seed=T, atlas_size=2048)
    frame.visible = (np.random.default_rng(T).uniform(size=T) < 0.6).astype(np.uint8)
    frame.visible[-1] = T % 2
    V = frame.num_vertices
    print(f"[gpu] prologue T={T} shift={shift}", flush=True)
    ctx = fa.Context(T, V, max_charts=16384, max_atlas=2048, tuning_table=None)
    out = ctx.outputs(fa.Mesh(frame.positions, frame.indices, 5), 2048)
    vis = torch.zeros(T + 4, dtype=torch.uint8, device="cuda")[shift:shift + T]
    vis.copy_(torch.as_tensor(frame.visible))
    out.chart_of_tri = torch.zeros(T + 4, dtype=torch.int32, device="cuda")[shift:shift + T]
    out.chart_of_vert = torch.zeros(V + 4, dtype=torch.int32, device="cuda")[shift:shift + V]
    ctx.build_atlas(fa.Mesh(frame.positions, frame.indices, 5), vis, frame.view_proj, frame.width,
                    frame.height, 2048, frame.rate, out=out)
    torch.cuda.synchronize()
    g = out.to_numpy()
    ctx.close()
    compare(g, oracle.build_frame(frame))


# A size outside [0, 2^24] ends the call before the push, in the order of one
# workgroup (up to 2048 boxes) and of several; the context goes on to pack.
@pytest.mark.parametrize("n", [1, 2048, 2049, 20000])
@pytest.mark.parametrize("bad", [-1.0, float("nan"), float("inf"), 16777218.0])
def test_refused_sizes(n, bad):
    fa = _fa()
    sizes = _uniform(n, 1, 8).astype(np.float32)
    ctx = fa.Context(1, 1, max_charts=65536, max_atlas=8192)
    for at in (0, n - 1):
        wrong = sizes.copy()
        wrong[at, at % 2] = bad
        print(f"[gpu] refused n={n} {bad} at {at}", flush=True)
        _, meta, cand = ctx.pack_boxes(torch.as_tensor(wrong).cuda(), 2048)
        m = fa.parse_meta(meta)
        assert m["status"] == fa.FA_ERR_INVALID_ARG and m["num_charts"] == n
        assert m["chosen_j"] == 0 and m["layout_width"] == 0
        assert not cand.cpu().numpy().any()
    sizes[0] = 16777216.0, 0.0
    _, meta, _ = ctx.pack_boxes(torch.as_tensor(sizes).cuda(), 2048)
    assert fa.parse_meta(meta)["status"] in (fa.FA_OK, fa.FA_ERR_NOFIT)
    ctx.close()


# The adjacency is built by ranges of vertices matched in LDS; meshes with a
# range of more than 4096 half-edges (a vertex of many triangles) or without
# room in the context's scratch are sorted instead. Tiles hold 2048 triangles.
def _fan_mesh(n):
    rim = np.arange(n)
    return np.stack([np.zeros(n, np.int64), 1 + rim, 1 + (rim + 1) % n], 1)


def _strip_mesh(n):
    i = np.arange(n)
    return np.stack([i, i + 1, i + 2], 1)


def _soup(n, V, seed):
    return np.random.default_rng(seed).integers(0, V, (n, 3))


ADJACENCY = {
    "one triangle": np.array([[0, 1, 2]]),
    "one vertex": np.zeros((5, 3), np.int64),
    "same triangle four times": np.tile([[4, 2, 7]], (4, 1)),
    "both windings": np.array([[0, 1, 2], [2, 1, 0], [0, 1, 3], [1, 0, 0]]),
    "2047 triangles": _strip_mesh(2047),
    "2049 triangles": _strip_mesh(2049),
    "fan of 1300": _fan_mesh(1300),             # 2600 half-edges meet at vertex 0
    "fan of 2100": _fan_mesh(2100),             # 4200: above a bucket
    "fan of 60000": _fan_mesh(60000),
    "few of many vertices": 1_000_000 + _soup(7000, 300, 1),
    "soup": _soup(20000, 9000, 2),
    "edges of many triangles": _soup(6000, 12, 3),
    "last vertices": 49_990 + _soup(3000, 10, 4),
}


@pytest.mark.parametrize("name", list(ADJACENCY))
def test_adjacency_ways(name):
    fa = _fa()
    idx = ADJACENCY[name].astype(np.int32)
    V = int(idx.max()) + 1
    print(f"[gpu] adjacency {name} T={len(idx)} V={V}", flush=True)
    ctx = fa.Context(len(idx), V, max_charts=16, max_atlas=16)
    mesh = fa.Mesh(np.zeros((V, 3), np.float32), idx, 5)
    want = oracle.adjacency(idx)
    for _ in range(2):  # a scene that comes back is built anew
        nbr = ctx.adjacency(mesh)
        torch.cuda.synchronize()
        assert np.array_equal(nbr.cpu().numpy(), want)
        assert fa.fa_scene_evict(ctx.h, 5) == fa.FA_OK
    bad = idx.copy()
    bad[-1, 1] = V
    for value in (V, -1):
        bad[-1, 1] = value
        with pytest.raises(fa.FastAtlasError) as e:
            ctx.adjacency(fa.Mesh(np.zeros((V, 3), np.float32), bad, 6))
        assert e.value.code == fa.FA_ERR_INVALID_ARG
    ctx.close()


# Meshes of up to 8192 triangles and 16384 vertices have their charts built by
# one workgroup (2 triangles a thread up to 2048 of them); larger ones by the
# tiled union-find.
@pytest.mark.parametrize("n", [1, 63, 64, 1023, 1025, 2048, 2049, 4000, 8191, 8192, 8193])
@pytest.mark.parametrize("per", [1, 5])
def test_front_sizes(n, per):
    rng = np.random.default_rng(n)
    owners = np.sort(rng.integers(0, max(1, n // per), n)) if per > 1 else np.arange(n)
    f = fans(np.unique(owners, return_inverse=True)[1], seed=n, atlas_size=2048)
    f.visible = (rng.uniform(size=n) < 0.7).astype(np.uint8)
    f.visible[rng.integers(n)] = 1
    compare(check(f), oracle.build_frame(f))


@pytest.mark.parametrize("V", [16384, 16385])
def test_front_vertices(V):
    # a strip over V vertices (the triangles wrap around it): long chains of
    # triangles in shuffled order
    rng = np.random.default_rng(V)
    t = rng.permutation(8000) * V // 8000
    f = fans(np.zeros(1, np.int64))
    pos = np.zeros((V, 3), np.float32)
    pos[:, 0] = np.linspace(-0.9, 0.9, V)
    pos[:, 1] = 0.4 * (-1.0) ** np.arange(V)
    idx = np.stack([t % V, (t + 1) % V, (t + 2) % V], 1).astype(np.int32)
    f.positions, f.indices = pos, idx
    f.visible = (rng.uniform(size=len(idx)) < 0.9).astype(np.uint8)
    f.name = f"strip/{V}"
    compare(check(f), oracle.build_frame(f))


def test_front_over_capacity():
    f = fans(np.repeat(np.arange(40), 2))
    fa = _fa()
    ctx = fa.Context(f.num_triangles, f.num_vertices, max_charts=32, max_atlas=1024)
    print("[gpu] 40 charts, capacity 32", flush=True)
    out = ctx.build_atlas(fa.Mesh(f.positions, f.indices, 3), torch.as_tensor(f.visible).cuda(),
                          f.view_proj, f.width, f.height, 1024, 1.0)
    torch.cuda.synchronize()
    m = out.to_numpy()["meta"]
    ctx.close()
    assert m["status"] == fa.FA_ERR_CAPACITY and m["num_charts"] == 40


# Edge-connected charts join tiles of consecutive visible triangles in LDS and
# look for a neighbour where it is if nothing in between is hidden: grids whose
# visible lists end around a tile, with none, a few and most triangles hidden.
@pytest.mark.parametrize("tile", [2048, 4096, 8192])
@pytest.mark.parametrize("count", [1, 2047, 2048, 2049, 8191, 8193, 20000])
@pytest.mark.parametrize("hidden", [0.0, 0.02, 0.8])
def test_edge_tiles(tile, count, hidden):
    fa = _fa()
    n = max(2, int(np.ceil(np.sqrt(count / (1.0 - hidden) / 2))) + 2)
    y, x = np.mgrid[0:n + 1, 0:n + 1] / n * 2 - 1
    pos = np.stack([x, y, 0.2 * np.sin(9 * x) * np.cos(7 * y)], -1).reshape(-1, 3)
    v = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).reshape(-1)
    tris = np.stack([v, v + 1, v + n + 2, v, v + n + 2, v + n + 1], 1).reshape(-1, 3)
    T = len(tris)
    rng = np.random.default_rng(count)
    keep = np.flatnonzero(rng.uniform(size=T) >= hidden)[:count]
    vis = np.zeros(T, np.uint8)
    vis[keep] = 1
    cam = scenes.make_camera((0.0, 0.0, 2.5), (0.0, 0.0, 0.0), 1280, 720, 0.05, 100.0, up=(0, 1, 0))
    f = scenes.Frame(f"edge tiles {count}", pos.astype(np.float32), tris.astype(np.int32), vis,
                     cam.view_proj, 1280, 720, 2048, 1.0, 994, cam.eye, cam.near, 0)
    print(f"[gpu] {f.name} hidden={hidden} tile={tile}", flush=True)
    ctx = fa.Context(T, len(pos), max_charts=65536, max_atlas=2048, flags=2, tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_UF_TILE, tile)
    out = ctx.build_atlas(fa.Mesh(f.positions, f.indices, 994), torch.as_tensor(vis).cuda(),
                          f.view_proj, 1280, 720, 2048, 1.0)
    torch.cuda.synchronize()
    g = out.to_numpy()
    ctx.close()
    r = oracle.build_frame(f, edge_only=True)
    assert g["meta"]["status"] == r["status"] and g["meta"]["num_charts"] == r["num_charts"]
    assert np.array_equal(g["chart_of_tri"], r["chart_of_tri"])
    assert np.array_equal(g["charts"]["root_tri"], r["roots"])


# A batch of 16 views on their slots' streams, half of them with everything
# visible, against the same frames alone. (One launch for all views, whose kernels
# then take several turns, is tested against the oracle with the other limits.)
def test_batch_turns():
    fa = _fa()
    n = 400
    y, x = np.mgrid[0:n + 1, 0:n + 1] / n * 2 - 1
    pos = np.stack([x, y, 0.2 * np.sin(9 * x) * np.cos(7 * y)], -1).reshape(-1, 3)
    v = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).reshape(-1)
    tris = np.stack([v, v + 1, v + n + 2, v, v + n + 2, v + n + 1], 1).reshape(-1, 3)
    T, V = len(tris), len(pos)
    mesh = fa.Mesh(pos.astype(np.float32), tris.astype(np.int32), 993)
    cams = [scenes.make_camera((0.3 * k - 2, 0.2 * k - 1, 2.0 + 0.1 * k), (0.0, 0.0, 0.0), 640, 360,
                               0.05, 100.0, up=(0, 1, 0)) for k in range(16)]
    rng = np.random.default_rng(4)
    vis = [torch.as_tensor((rng.uniform(size=T) < (1.0 if k % 2 else 0.1 * k)).astype(np.uint8)
                           ).cuda() for k in range(16)]
    ctx = fa.Context(T, V, max_charts=65536, max_atlas=1024, max_views=16, tuning_table=None)
    print("[gpu] batch of 16 views", flush=True)
    outs = [ctx.outputs(mesh, 1024) for _ in cams]
    ctx.build_atlas_batch(mesh, [(a, c.view_proj, 640, 360, 1024, 1.0) for a, c in zip(vis, cams)],
                          outs)
    torch.cuda.synchronize()
    for a, c, o in zip(vis, cams, outs):
        alone = ctx.build_atlas(mesh, a, c.view_proj, 640, 360, 1024, 1.0)
        torch.cuda.synchronize()
        g, h = o.to_numpy(), alone.to_numpy()
        assert g["meta"] == h["meta"]
        for k in ("chart_of_tri", "chart_of_vert", "occupancy", "candidates", "charts"):
            assert np.array_equal(g[k], h[k]), k
        assert np.array_equal(g["uv"].view(np.uint32), h["uv"].view(np.uint32))
    ctx.close()
