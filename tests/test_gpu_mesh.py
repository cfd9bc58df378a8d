"""Triangle-mesh bodies on the GPU against the FP64 oracle: the FP16 distance
grid built on the mesh, and path-by-path renders (plain tracing, sphere
tracing with exact in-sphere walks and with BF16 learned steps) through the
stackless BVH."""
import numpy as np
import pytest
import torch

import workloads as W
from conftest import announce
from test_gpu_render import CVAE, EXACT, LEARNED_REL, PLAIN, ST, compare_paths, f32_camera, f32_light, f32_medium, \
    models_for_test, pack_all

pytestmark = pytest.mark.gpu

LO, HI = (-1.2, -1.2, -1.2), (1.2, 1.2, 1.2)


@pytest.fixture(scope="module")
def blob():
    return W.mesh_blob(0, 3)


def test_mesh_grid_matches_oracle(msst, oracle, blob):
    announce("mesh sdf grid")
    res = 32
    g = msst.build_sdf_grid(None, res, LO, HI, tris=blob).cpu().numpy().view(np.uint16)
    o = oracle.Scene(None, tris=blob).build_grid(res, LO, HI)
    diff = np.abs(g.astype(np.int64) - o.astype(np.int64))
    gv, ov = g.view(np.float16).astype(np.float64), o.view(np.float16).astype(np.float64)
    print(f"exact {(diff == 0).mean():.5f}, max diff {diff.max()}, inside {(ov < 0).mean():.3f}")
    assert (diff == 0).mean() > 0.999 and diff.max() <= 1
    assert np.all(np.sign(gv) * np.sign(ov) >= 0)


@pytest.mark.parametrize("method,sampler", [(PLAIN, CVAE), (ST, EXACT), (ST, CVAE)])
def test_mesh_render_path_by_path(msst, oracle, blob, method, sampler):
    announce(f"mesh render method={method} sampler={sampler}")
    res = 64
    grid_g = msst.build_sdf_grid(None, res, LO, HI, tris=blob)
    grid_o = oracle.Scene(None, tris=blob).build_grid(res, LO, HI)
    cam, light = f32_camera(W.camera_mesh(40, 40)), f32_light(W.light_c4())
    med = f32_medium(W.medium_c4(20.0))
    opts = dict(spp=1, seed=31)
    kw_o = dict(method=oracle.METHOD_PLAIN_NEE if method == PLAIN else oracle.METHOD_ST)
    packed = (None, None, None)
    if method == ST:
        opts["tau_min"] = 2.0
        kw_o["sampler"] = oracle.SAMPLER_EXACT_WALK if sampler == EXACT else oracle.SAMPLER_CVAE
        if sampler == CVAE:
            models, src = models_for_test(oracle)
            packed = pack_all(msst, src, 1)
            opts.update(nee_samples=2, flags=1)
            kw_o.update(models=models, precision=oracle.PREC_BF16)
    r = msst.Renderer(None, cam, light, grid=grid_g, grid_lo=LO, grid_hi=HI, tris=blob)
    out = r.render(med, method=method, sampler=sampler, packed=packed, **opts)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in out.items()}
    o = oracle.render(oracle.Scene(None, sdf_fp16=grid_o, lo=LO, hi=HI, tris=blob), cam, light, med, **kw_o, **opts)
    frac, _ = compare_paths(g, o, rel=LEARNED_REL)
    print(f"diverged {frac:.2e}; lit {(o['sum'] > 0).mean():.2f}, events {o['events'].sum()}, steps {o['steps'].sum()}")
    assert (o["sum"] > 0).mean() > 0.1
    assert frac < 2e-3
    if method == ST:
        assert o["steps"].sum() > 50


def thin_triangles(seed, n):
    """An open soup of triangles, a third of them needles and a seventh
    without area: no filter may drop one, nor take a bound from one."""
    rng = np.random.default_rng(seed)
    t = (0.4 * rng.normal(size=(n, 9))).astype(np.float32)
    t[::3, 6:9] = t[::3, 3:6] + (1e-6 * rng.normal(size=t[::3, 3:6].shape)).astype(np.float32)
    t[::7, 3:6] = t[::7, 0:3]
    return t


@pytest.mark.parametrize("name,res", [("coarse", 1), ("coarse", 5), ("fine", 9), ("fine", 16), ("thin", 18),
                                      ("one", 7), ("many", 6)])
def test_mesh_grid_culling_matches_oracle(msst, oracle, name, res):
    """The grid at the edges of its bricks (sizes around multiples of four),
    with lists of one part (80 triangles) and of several (20 480 triangles,
    all kept around the centre; 6 000 overlapping needles), one triangle, and
    triangles too thin for FP32.  Both sides evaluate the same FP64 distance
    and crossing of every triangle that matters, so a voxel differs only where
    the two compilers' FP64 rounding (1e-16 relative) straddles a binary16
    step (1e-3): none of these few thousand is expected to."""
    announce(f"mesh sdf grid culling {name} res={res}")
    tris = {"coarse": lambda: W.mesh_blob(1, 1), "fine": lambda: W.mesh_blob(2, 5),
            "thin": lambda: thin_triangles(3, 300), "one": lambda: W.mesh_blob(0, 0)[:1],
            "many": lambda: thin_triangles(4, 6000)}[name]()
    g = msst.build_sdf_grid(None, res, LO, HI, tris=tris).cpu().numpy().view(np.uint16)
    o = oracle.Scene(None, tris=tris).build_grid(res, LO, HI)
    assert np.array_equal(g, o), (int((g != o).sum()), g.size)


def sheets_beside_large_triangles(seed, size):
    """Three triangles of `size`, their centroids within the grid, each with a
    finely tessellated sheet 2e-8 of its size beside its plane: on one side of
    the pair the large triangle is the nearest by less than FP32 resolves at
    its vertices."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(3):
        q = np.linalg.qr(rng.normal(size=(3, 3)))[0]
        ang = rng.uniform(0, 2 * np.pi) + np.arange(3) * 2 * np.pi / 3
        big = (rng.uniform(-0.5, 0.5, 3) + size * (np.cos(ang)[:, None] * q[0] + np.sin(ang)[:, None] * q[1])).astype(np.float32)
        v = big.astype(np.float64)
        nrm = np.cross(v[1] - v[0], v[2] - v[0])
        nrm /= np.linalg.norm(nrm)
        e = v[1] - v[0]
        e /= np.linalg.norm(e)
        f = np.cross(nrm, e)
        u = np.linspace(-0.8, 0.8, 21)
        p = (v.mean(0) + 2e-8 * size * nrm + u[:, None, None] * e + u[None, :, None] * f).astype(np.float32)
        quads = p[:-1, :-1], p[1:, :-1], p[1:, 1:], p[:-1, 1:]
        out += [big.reshape(1, 9)]
        for k in ((0, 1, 2), (0, 2, 3)):
            out.append(np.concatenate([quads[j] for j in k], -1).reshape(-1, 9))
    return np.concatenate(out)


@pytest.mark.parametrize("size", [1e2, 1e3, 1e4, 1e6])
def test_mesh_grid_beside_large_triangles_matches_oracle(msst, oracle, size):
    """Triangles that reach far beyond the grid: their FP32 centroids and
    distances are off by their vertices' rounding, which must neither drop a
    triangle nor bound the distance too tightly.  As above both sides evaluate
    the same FP64 distances; their rounding (1e-16 of the size, 1e-10 at most)
    straddles a binary16 step (6e-5 or more at the distances of all but a
    hundredth of the voxels) for one voxel in 10^6."""
    announce(f"mesh sdf grid beside triangles of {size:g}")
    tris = sheets_beside_large_triangles(int(size) % 97, size)
    g = msst.build_sdf_grid(None, 20, LO, HI, tris=tris).cpu().numpy().view(np.uint16)
    o = oracle.Scene(None, tris=tris).build_grid(20, LO, HI)
    d = np.abs(g.view(np.float16).astype(np.float64)) - np.abs(o.view(np.float16).astype(np.float64))
    assert np.array_equal(g, o), (int((g != o).sum()), g.size, float(d.max()))
