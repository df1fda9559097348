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
