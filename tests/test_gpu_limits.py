"""Frames, batches and scenes at the limits of the library's dispatch: frames
that end without a packing or over a capacity, indices that no scene has
checked, batches whose views need several turns of their workgroups."""
import numpy as np
import pytest
import torch

import oracle
from synth import scenes
from test_gpu_dispatch import fans
from test_gpu_parity import _fa, compare

pytestmark = pytest.mark.gpu


def _poison(o):
    for t in (o.chart_of_tri, o.chart_of_vert, o.occupancy, o.candidates, o.charts, o.meta):
        t.fill_(-7)
    o.uv.fill_(-7.0)


# A frame that fits at no scale places nothing, however many workgroups the
# placement has (256 charts each): the placement words of the chart records keep
# what they held, the map is empty and no vertex is mapped. One frame, views of
# a batch on streams and in one launch, and boxes alone.
@pytest.mark.parametrize("n", [256, 257, 3000, 20000])
def test_no_fit_places_nothing(n):
    fa = _fa()
    f = fans(np.arange(n), seed=n, atlas_size=16)
    want = oracle.build_frame(f)
    assert want["status"] == oracle.STATUS_NOFIT
    ctx = fa.Context(f.num_triangles, f.num_vertices, max_charts=32768, max_atlas=64, max_views=3,
                     tuning_table=None)
    mesh = fa.Mesh(f.positions, f.indices, 3)
    vis = torch.as_tensor(f.visible).cuda()
    for way in ("frame", "streams", "one launch"):
        print(f"[gpu] no fit, {n} charts, {way}", flush=True)
        outs = [ctx.outputs(mesh, 16) for _ in range(1 if way == "frame" else 3)]
        for o in outs:
            _poison(o)
        if way == "frame":
            ctx.build_atlas(mesh, vis, f.view_proj, f.width, f.height, 16, 1.0, out=outs[0])
        else:
            ctx.set_tuning(fa.FA_TUNE_BATCH_LAUNCH, int(way == "one launch"))
            ctx.build_atlas_batch(mesh, [(vis, f.view_proj, f.width, f.height, 16, 1.0)] * 3, outs)
        torch.cuda.synchronize()
        for o in outs:
            g = o.to_numpy()
            compare(g, want)
            assert g["meta"]["occupied_texels"] == 0 and g["meta"]["layout_width"] == 0
            for k in ("x", "y", "w", "h"):
                assert (g["charts"][k] == -7).all(), k
            assert (g["occupancy"] == -1).all() and np.isnan(g["uv"]).all()
    print(f"[gpu] no fit, {n} boxes", flush=True)
    sizes = torch.as_tensor(np.ascontiguousarray(want["target"], np.float32)).cuda()
    meta = torch.zeros(16, dtype=torch.int32, device="cuda")
    cand = torch.zeros((64, 4), dtype=torch.int32, device="cuda")
    placed = torch.full((n, 5), -7, dtype=torch.int32, device="cuda")
    assert fa.fa_pack_boxes(ctx.h, sizes.data_ptr(), n, 16, placed.data_ptr(), meta.data_ptr(),
                            cand.data_ptr(), torch.cuda.current_stream().cuda_stream) == fa.FA_OK
    torch.cuda.synchronize()
    assert fa.parse_meta(meta)["status"] == fa.FA_ERR_NOFIT
    assert (placed == -7).all().item()
    assert np.array_equal(cand.cpu().numpy()[:, :3], want["cand"][:, :3])
    ctx.close()


# A frame of more charts than the context holds ends with FA_ERR_CAPACITY and the
# whole count; the roots of the charts below the capacity are labelled, whichever
# workgroups (1024 visible triangles each) start after the last one reports it.
@pytest.mark.parametrize("n,cap,static", [
    (8192, 1, False), (8193, 8192, False), (60000, 700, False), (60000, 59999, False),
    (8192, 4096, True), (20000, 4096, True)])
def test_over_capacity_labels(n, cap, static):
    fa = _fa()
    f = fans(np.arange(n), seed=n, atlas_size=64)
    print(f"[gpu] {n} charts, capacity {cap}, static={static}", flush=True)
    mesh = fa.Mesh(f.positions, f.indices, 4)
    vis = torch.as_tensor(f.visible).cuda()
    out = fa.AtlasOutputs(n, f.num_vertices, cap, 64, 64)
    _poison(out)
    ctx = None
    if static:
        fa.build_atlas_static(mesh, vis, f.view_proj, f.width, f.height, 64, 1.0, out=out)
    else:
        ctx = fa.Context(n, f.num_vertices, max_charts=cap, max_atlas=64, tuning_table=None)
        ctx.build_atlas(mesh, vis, f.view_proj, f.width, f.height, 64, 1.0, out=out)
    torch.cuda.synchronize()
    m = fa.parse_meta(out.meta)
    assert m["status"] == fa.FA_ERR_CAPACITY and m["num_charts"] == n
    label = np.where(np.arange(n) < cap, np.arange(n), -1)  # (every triangle is a root)
    assert np.array_equal(out.chart_of_tri.cpu().numpy(), label)
    assert np.array_equal(fa.parse_charts(out.charts, cap)["root_tri"], np.arange(cap))
    assert (out.occupancy == -1).all().item() and torch.isnan(out.uv).all().item()
    if ctx is not None:
        ctx.close()


# A batch in one launch per stage limits the workgroups of its views: with 16
# views a turn holds 131072 list entries of the vertex hook and of the raster and
# 262144 of the box gather, whose table of charts then serves all its turns. Odd
# views show 320000 triangles, even ones fewer; one chart (a sheet) and 10000
# (the sheet cut into squares of 4 x 4 cells).
@pytest.mark.parametrize("square", [400, 4])
def test_one_launch_batch_takes_turns(square):
    fa = _fa()
    n, k = 400, 400 // square
    cell = np.arange(square + 1) / square
    at = (np.stack(np.meshgrid(np.arange(k), np.arange(k), indexing="ij"), -1).reshape(-1, 1, 1, 2)
          + 0.98 * np.stack(np.meshgrid(cell, cell, indexing="ij"), -1)) / k * 2 - 1
    y, x = at[..., 0], at[..., 1]
    pos = np.stack([x, y, 0.2 * np.sin(9 * x) * np.cos(7 * y)], -1).reshape(-1, 3)
    s1 = square + 1
    v = (np.arange(square)[:, None] * s1 + np.arange(square)).reshape(-1)
    quad = np.stack([v, v + 1, v + s1 + 1, v, v + s1 + 1, v + s1], 1).reshape(-1, 3)
    tris = (np.arange(k * k)[:, None, None] * s1 * s1 + quad).reshape(-1, 3)
    assert len(tris) == 2 * n * n
    pos, tris = pos.astype(np.float32), tris.astype(np.int32)
    rng = np.random.default_rng(square)
    views = []
    for i in range(16):
        cam = scenes.make_camera((0.1 * i - 0.8, 0.7 - 0.1 * i, 2.0 + 0.1 * i), (0.0, 0.0, 0.0), 640,
                                 360, 0.05, 100.0, up=(0, 1, 0))
        vis = (rng.uniform(size=len(tris)) < (1.0 if i % 2 else 0.06 * i)).astype(np.uint8)
        views.append(scenes.Frame(f"turns/{square}/{i}", pos, tris, vis, cam.view_proj, 640, 360,
                                  1024, 1.0 + 0.1 * i, 995, cam.eye, cam.near, 0))
    ctx = fa.Context(len(tris), len(pos), max_charts=65536, max_atlas=1024, max_views=16,
                     tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_BATCH_LAUNCH, 1)
    assert ctx.get_tuning(fa.FA_TUNE_BATCH_LAUNCH) == 1
    mesh = fa.Mesh(pos, tris, 995)
    outs = [ctx.outputs(mesh, 1024) for _ in views]
    for o in outs:
        _poison(o)
    shown = [torch.as_tensor(f.visible).cuda() for f in views]
    print(f"[gpu] 16 views in one launch, squares of {square}", flush=True)
    ctx.build_atlas_batch(mesh, [(a, f.view_proj, 640, 360, 1024, f.rate)
                                 for a, f in zip(shown, views)], outs)
    torch.cuda.synchronize()
    for o, f in zip(outs, views):
        compare(o.to_numpy(), oracle.build_frame(f))
    ctx.close()


# Small meshes have their charts built by one workgroup a view in a batch too: two
# triangles a thread up to 2048 of them and eight above; views of uneven atlas
# sizes that show nothing, some and all of the mesh.
@pytest.mark.parametrize("n", [1, 64, 1025, 2048, 2049, 8192])
def test_small_mesh_batch(n):
    fa = _fa()
    rng = np.random.default_rng(n)
    owners = np.unique(np.sort(rng.integers(0, max(1, n // 3), n)), return_inverse=True)[1]
    base = fans(owners, seed=n)
    views = []
    for i, omega in enumerate((64, 2048, 256, 1024, 512)):
        vis = (rng.uniform(size=n) < (0.0, 1.0, 0.5, 0.9, 0.1)[i]).astype(np.uint8)
        views.append(scenes.Frame(f"{base.name}/{i}", base.positions, base.indices, vis,
                                  base.view_proj, base.width, base.height, omega, 0.7, 996,
                                  base.eye, base.near, 0))
    ctx = fa.Context(n, base.num_vertices, max_charts=4096, max_atlas=2048, max_views=3,
                     tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_BATCH_LAUNCH, 1)
    mesh = fa.Mesh(base.positions, base.indices, 996)
    outs = [ctx.outputs(mesh, f.atlas_size) for f in views]
    for o in outs:
        _poison(o)
    shown = [torch.as_tensor(f.visible).cuda() for f in views]
    print(f"[gpu] 5 views of {n} triangles on 3 slots", flush=True)
    ctx.build_atlas_batch(mesh, [(a, f.view_proj, f.width, f.height, f.atlas_size, f.rate)
                                 for a, f in zip(shown, views)], outs)
    torch.cuda.synchronize()
    for o, f in zip(outs, views):
        compare(o.to_numpy(), oracle.build_frame(f))
    ctx.close()


# The allocation-free entry point checks the indices itself. Meshes above 8192
# triangles or 16384 vertices do it by tiles of 1024 triangles, four a workgroup,
# and the compaction of the last tile ends the frame: bad indices at each of a
# workgroup's tiles, in the first, inner and last (full or partial) tile, of
# hidden triangles, and of all triangles at once; then a good frame.
@pytest.mark.parametrize("T,spare", [(8193, 0), (21504, 0), (20001, 1000), (5000, 12000)])
def test_static_index_check_in_tiles(T, spare):
    fa = _fa()
    f = fans(np.arange(T) // 8, seed=T, atlas_size=512)
    f.positions = np.concatenate([f.positions, np.zeros((spare, 3), np.float32)])
    V = f.num_vertices
    assert V <= fa.STATIC_MAX_VERTICES and (T > 8192 or V > 16384)
    want = oracle.build_frame(f)
    mesh = fa.Mesh(f.positions, f.indices, 5)
    out = fa.AtlasOutputs(T, V, fa.STATIC_MAX_CHARTS, 512, 64)
    hidden = f.visible.copy()
    hidden[::3] = 0
    where = [0, 1023, 1024, 2049, 3072 + 3, 4096, T // 2, T - 1, slice(None),
             slice((T - 1) // 1024 * 1024, T)]
    for k, at in enumerate(where):
        idx = f.indices.copy()
        idx[at, k % 3] = (V, -1, 2**31 - 1, -2**31)[k % 4]
        vis = torch.as_tensor(hidden if k % 2 else f.visible).cuda()
        print(f"[gpu] static: T={T} V={V}, bad index at {at}", flush=True)
        _poison(out)
        fa.build_atlas_static(fa.Mesh(f.positions, idx, 6), vis, f.view_proj, f.width, f.height,
                              512, f.rate, out=out)
        torch.cuda.synchronize()
        m = fa.parse_meta(out.meta)
        assert m["status"] == fa.FA_ERR_INVALID_ARG, at
        assert m["visible_triangles"] == 0 and m["num_charts"] == 0 and m["chosen_j"] == 0, at
    _poison(out)
    fa.build_atlas_static(mesh, torch.as_tensor(f.visible).cuda(), f.view_proj, f.width, f.height,
                          512, f.rate, out=out)
    torch.cuda.synchronize()
    compare(out.to_numpy(), want)


# Meshes of more buckets than the adjacency's vertex ranges have, and those whose
# half-edges do not fit the context's scratch, are sorted, and their indices
# checked by a kernel of its own: good ones against the oracle, bad ones (at the
# ends and inside) refused.
@pytest.mark.parametrize("T,V", [(2_810_000, 8200), (5_600_000, 8000)])
def test_adjacency_of_large_meshes(T, V):
    fa = _fa()
    idx = np.random.default_rng(T).integers(0, V, (T, 3), dtype=np.int32)
    ctx = fa.Context(T, V, max_charts=16, max_atlas=16)
    pos = np.zeros((V, 3), np.float32)
    print(f"[gpu] sorted adjacency T={T} V={V}", flush=True)
    nbr = ctx.adjacency(fa.Mesh(pos, idx, 5))
    torch.cuda.synchronize()
    assert np.array_equal(nbr.cpu().numpy(), oracle.adjacency(idx))
    for at, value in (((0, 0), V), ((T - 1, 2), -1), ((T // 2, 1), 2**31 - 1)):
        bad = idx.copy()
        bad[at] = value
        print(f"[gpu] sorted adjacency T={T}, index {value} at {at}", flush=True)
        with pytest.raises(fa.FastAtlasError) as e:
            ctx.adjacency(fa.Mesh(pos, bad, 6))
        assert e.value.code == fa.FA_ERR_INVALID_ARG
    ctx.close()


def test_device_bytes_count_the_check_words():
    # what a context holds: scratch parts and view descriptors, all multiples of
    # 256 bytes, and the two words of the index check
    fa = _fa()
    for T, V, views in ((1, 1, 1), (1000, 777, 3), (70001, 30001, 2)):
        ctx = fa.Context(T, V, max_charts=100, max_atlas=64, max_views=views)
        print(f"[gpu] device bytes T={T} V={V} views={views}", flush=True)
        assert ctx.device_bytes() % 256 == 8
        ctx.close()


# The box push goes by rows or by columns, whichever is estimated to take less
# from the rows, the boxes' widths and how many lie over edge columns: sets on
# either side and around the line, of one chunk and of several, with more boxes
# over edge columns than a row's table holds.
def _mixed(n, mean, aspect, share, factor, seed):
    rng = np.random.default_rng(seed)
    z = rng.lognormal(0, 0.3, (n, 2)) * np.array([aspect ** 0.5, aspect ** -0.5])
    k = max(1, int(n * share))
    z[:k] = rng.lognormal(0, 0.3, (k, 2)) * factor
    return (rng.permutation(z) * mean / np.sqrt((z[:, 0] * z[:, 1]).mean())).astype(np.float32)


PUSH_WAYS = {
    "rows, many over edges": (_mixed(4000, 40, 1.0, 0.01, 10, 1), 4096),
    "rows, several chunks, many over edges": (_mixed(20000, 20, 0.25, 0.01, 10, 2), 4096),
    "columns, narrow boxes": (_mixed(20000, 13, 0.06, 0.01, 1, 3), 4096),
    "columns, narrow with wide": (_mixed(16000, 5, 1.0, 0.01, 30, 4), 1024),
    "columns, several chunks, with wide": (_mixed(16000, 20, 0.25, 0.01, 30, 5), 4096),
    "few boxes": (_mixed(20, 100, 1.0, 0.1, 3, 6), 1024),
    "around the line": (_mixed(1000, 20, 1.0, 0.01, 10, 7), 1024),
}


@pytest.mark.parametrize("name", list(PUSH_WAYS))
@pytest.mark.parametrize("block", [256, 512, 1024])
def test_push_ways(name, block):
    from test_gpu_parity import _oracle_pack
    fa = _fa()
    sizes, omega = PUSH_WAYS[name]
    print(f"[gpu] push {name} n={len(sizes)} omega={omega} block={block}", flush=True)
    ctx = fa.Context(1, 1, max_charts=32768, max_atlas=4096, num_scales=16, tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_PACK_BLOCK, block)
    placed, meta, cand = ctx.pack_boxes(torch.as_tensor(sizes).cuda(), omega)
    torch.cuda.synchronize()
    m, c = fa.parse_meta(meta), cand.cpu().numpy()
    placed = placed.cpu().numpy()
    ctx.close()
    js, table, want = _oracle_pack(sizes, omega, 16, 1, 2)
    assert js > 0 and m["chosen_j"] == js and np.array_equal(placed, want)
    assert np.array_equal(c[:, :3], table[:, :3])
    fit = table[:, 0] == 1
    assert np.array_equal(c[fit, 3], table[fit, 3])
    assert ((c[~fit, 3] == -1) | (c[~fit, 3] > c[~fit, 2])).all()


# Union-find modes 0 and 1 start every visible triangle at its smallest visible
# neighbour, four triangles a lane and a tile of 1024 a workgroup: sizes around
# those, neighbours hidden or not, visible buffers of any alignment, and triangles
# that name an edge twice.
@pytest.mark.parametrize("T", [8193, 9215, 12291, 16384, 20002])
@pytest.mark.parametrize("hooks", [0, 1])
def test_linked_start(T, hooks):
    fa = _fa()
    n = int(np.ceil(np.sqrt(T / 2)))
    y, x = np.mgrid[0:n + 1, 0:n + 1] / n * 2 - 1
    pos = np.stack([x, y, 0.2 * np.sin(9 * x) * np.cos(7 * y)], -1).reshape(-1, 3)
    v = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).reshape(-1)
    tris = np.stack([v, v + 1, v + n + 2, v, v + n + 2, v + n + 1], 1).reshape(-1, 3)[:T]
    rng = np.random.default_rng(T + hooks)
    tris = tris[rng.permutation(T)] if T % 2 else tris
    tris[T // 3] = tris[T // 3][[0, 1, 0]]
    cam = scenes.make_camera((0.0, 0.0, 2.5), (0.0, 0.0, 0.0), 1280, 720, 0.05, 100.0, up=(0, 1, 0))
    ctx = fa.Context(T, len(pos), max_charts=16384, max_atlas=1024, tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_UF_EDGE_HOOKS, hooks)
    assert ctx.get_tuning(fa.FA_TUNE_UF_LINK_INIT) == 1
    mesh = fa.Mesh(pos, tris, 997)
    for shift, share in ((0, 1.0), (1, 0.6), (2, 0.3), (3, 0.02)):
        vis = (rng.uniform(size=T) < share).astype(np.uint8)
        f = scenes.Frame(f"linked {T}", pos.astype(np.float32), tris.astype(np.int32), vis,
                         cam.view_proj, 1280, 720, 1024, 1.0, 997, cam.eye, cam.near, 0)
        print(f"[gpu] linked start T={T} hooks={hooks} shift={shift}", flush=True)
        shown = torch.zeros(T + 4, dtype=torch.uint8, device="cuda")[shift:shift + T]
        shown.copy_(torch.as_tensor(vis))
        out = ctx.outputs(mesh, 1024)
        _poison(out)
        ctx.build_atlas(mesh, shown, f.view_proj, 1280, 720, 1024, 1.0, out=out)
        torch.cuda.synchronize()
        compare(out.to_numpy(), oracle.build_frame(f))
    ctx.close()


# Edge-connected charts over edges of more than two triangles: the visible ones of
# an edge are joined whichever of the others between them are hidden, in the global
# hook and in tiles; triangles that name an edge twice, and edges across tiles.
@pytest.mark.parametrize("kind", ["pages", "books", "soup"])
@pytest.mark.parametrize("hooks,tile", [(1, 2048), (5, 2048), (5, 4096), (5, 8192)])
def test_edge_charts_over_many_at_an_edge(kind, hooks, tile):
    fa = _fa()
    rng = np.random.default_rng(tile + hooks)
    if kind == "pages":    # all of them at one edge
        tris = np.stack([np.zeros(300, int), np.ones(300, int), 2 + np.arange(300)], 1)
    elif kind == "books":  # edges of 3 to 5 triangles, which lie all over the list
        k, n = 2500, rng.integers(3, 6, 2500)
        spine = np.repeat(np.arange(k), n)
        tris = np.stack([2 * spine, 2 * spine + 1, 2 * k + np.arange(len(spine))], 1)
        tris = tris[rng.permutation(len(tris))]
    else:
        tris = rng.integers(0, 400, (6000, 3))
    flip = rng.uniform(size=len(tris)) < 0.5
    tris[flip] = tris[flip][:, [1, 0, 2]]
    tris[7] = tris[7][[0, 1, 0]]
    V = int(tris.max()) + 1
    pos = rng.uniform(-1, 1, (V, 3)).astype(np.float32)
    cam = scenes.make_camera((0.0, 0.0, 3.0), (0.0, 0.0, 0.0), 640, 360, 0.05, 100.0, up=(0, 1, 0))
    ctx = fa.Context(len(tris), V, max_charts=16384, max_atlas=1024, flags=2, tuning_table=None)
    ctx.set_tuning(fa.FA_TUNE_UF_EDGE_HOOKS, hooks)
    ctx.set_tuning(fa.FA_TUNE_UF_TILE, tile)
    mesh = fa.Mesh(pos, tris, 998)
    for share in (0.05, 0.5, 0.9, 1.0):
        vis = (rng.uniform(size=len(tris)) < share).astype(np.uint8)
        f = scenes.Frame(f"{kind} {share}", pos, tris.astype(np.int32), vis, cam.view_proj, 640, 360,
                         1024, 0.25, 998, cam.eye, cam.near, 0)
        print(f"[gpu] edge charts, {kind}, hooks={hooks} tile={tile} shown {share}", flush=True)
        out = ctx.outputs(mesh, 1024)
        _poison(out)
        ctx.build_atlas(mesh, torch.as_tensor(vis).cuda(), f.view_proj, 640, 360, 1024, 0.25,
                        out=out)
        torch.cuda.synchronize()
        g, r = out.to_numpy(), oracle.build_frame(f, edge_only=True)
        assert g["meta"]["status"] == r["status"] and g["meta"]["num_charts"] == r["num_charts"]
        assert np.array_equal(g["chart_of_tri"], r["chart_of_tri"])
        assert np.array_equal(g["chart_of_vert"], r["chart_of_vert"])
        assert np.array_equal(g["charts"]["root_tri"], r["roots"])
    ctx.close()
