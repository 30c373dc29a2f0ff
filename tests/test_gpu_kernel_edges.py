"""Kernels at the sizes where a tile, a remainder or a dispatch rule can go
wrong: the smallest and largest of each range, one below and above a tile."""
import numpy as np
import pytest

from paper_2111_06906_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_2111_06906_amd import engine
    return engine


def _soup(n_tris, n_mat, counts, B, rng):
    """A static scene of small random triangles with random materials."""
    tri = (rng.uniform(-1, 1, (n_tris, 1, 3)) + rng.uniform(-0.01, 0.01, (n_tris, 3, 3))).astype(np.float32)
    L = len(counts)
    xf = np.tile(np.array([1, 0, 0, 0, 0, 0, -1, 0.9, 0, 1, 0, 0], np.float32), (1, L, 1))
    return scenes.Scene(
        name="soup", static_verts=tri, static_mat=rng.integers(0, n_mat, n_tris).astype(np.uint32), obj_local=[],
        obj_mat=[], obj_xforms=np.zeros((1, 0, 12), np.float32),
        albedo=rng.uniform(0.3, 0.8, (n_mat, 3)).astype(np.float32), light_half=np.full((L, 2), 0.05, np.float32),
        light_power=rng.uniform(0.5, 2.0, (L, 3)).astype(np.float32), light_xforms=xf,
        light_paths=np.asarray(counts, np.int64), max_bounces=B, threshold=0.01, seed=1)


def _random_store(E, ctx, sc, rng):
    """A store of random photons: hits anywhere in the scene, 0..B segments per path."""
    n, B = sc.n_paths, sc.max_bounces
    d = dict(pos=rng.uniform(-1, 1, (B, n, 3)).astype(np.float32),
             hit=rng.integers(0, sc.n_static, (B, n)).astype(np.uint32),
             energy=rng.uniform(0, 1, (B, n, 3)).astype(np.float32), radius=np.full((B, n), 0.01, np.float32),
             origin=rng.uniform(-1, 1, (n, 3)).astype(np.float32),
             info=(rng.integers(0, B + 1, n).astype(np.uint32) << 22))
    st = ctx.new_store()
    st.load_numpy(d)
    return st, d


# Gradients and energies: a lone path, one below / at / above a path tile, more
# tiles than the gradient grid holds workgroups, both row-array sizes (8, 15),
# every number of accumulator copies (2 .. 256 materials), a light without
# paths.  All terms are non-negative, so an energy (at most 15 FP32 products)
# is within 16 x 2^-24 and a gradient (per term at most 14 products, 2 x 14
# recurrence roundings and 4 more, summed in FP64) within 50 x 2^-24 of FP64.
@pytest.mark.parametrize("counts,B,n_mat", [
    ([1], 1, 1), ([255], 2, 3), ([256, 0], 8, 32), ([100, 157], 9, 80), ([200, 57, 300], 15, 256),
    ([150_000, 120_011], 7, 81), ([300_001], 4, 2)])
def test_energy_and_gradients_at_edges(E, counts, B, n_mat):
    import torch
    rng = np.random.default_rng(B * 1000 + n_mat)
    sc = _soup(500, n_mat, counts, B, rng)
    ctx = E.Context(sc)
    st, d = _random_store(E, ctx, sc, rng)
    n = sc.n_paths
    g = rng.uniform(0, 1, (B, n, 3)).astype(np.float32)
    alb, pw = torch.from_numpy(sc.albedo).cuda(), torch.from_numpy(sc.light_power).cuda()
    light = np.repeat(np.arange(len(counts)), counts)
    nseg = d["info"] >> 22
    rho = torch.from_numpy(sc.albedo).double().requires_grad_(True)
    phi = torch.from_numpy(sc.light_power).double().requires_grad_(True)
    e = rho.sum() * 0.0 + phi[light] / torch.from_numpy(np.asarray(counts, np.float64)[light])[:, None]
    rows = []
    for r in range(B):
        if r:
            e = e * rho[sc.static_mat[d["hit"][r - 1]].astype(np.int64)]
        rows.append(e * torch.from_numpy((nseg > r).astype(np.float64))[:, None])
    ref = torch.stack(rows)
    ref.backward(torch.from_numpy(g).double())
    got = ctx.energy_forward(st, alb, pw).cpu().numpy()
    np.testing.assert_allclose(got, ref.detach().numpy(), rtol=16 * 2.0 ** -24, atol=0)
    for _ in range(2):  # the second call starts from what the first one left
        ga, gp = ctx.energy_backward(st, alb, pw, torch.from_numpy(g).cuda())
        np.testing.assert_allclose(ga.cpu().numpy(), rho.grad.numpy(), rtol=50 * 2.0 ** -24, atol=0)
        np.testing.assert_allclose(gp.cpu().numpy(), phi.grad.numpy(), rtol=50 * 2.0 ** -24, atol=0)
    ctx.close()


# The four-wide walk gives up where it would leave more entries than the stack
# holds and where two crossings lie within rounding of each other; the binary
# walk then answers.


def _crowded(n_static, n_obj, frames=3):
    """The tiny box filled with large overlapping triangles, static ones and
    an object's: a ray enters nearly every box of both hierarchies, so walks
    leave as many entries as their trees allow."""
    sc = scenes.make_tiny(n_paths=2048 + 3, max_bounces=3, frames=frames, seed=21)
    rng = np.random.default_rng(21)
    st = rng.uniform(0.05, 0.95, (n_static, 3, 3)).astype(np.float32)
    ob = rng.uniform(-0.25, 0.25, (n_obj, 3, 3)).astype(np.float32)
    sc.static_verts = np.concatenate([sc.static_verts, st])
    sc.static_mat = np.concatenate([sc.static_mat, np.zeros(n_static, np.uint32)])
    sc.obj_local = [np.concatenate([sc.obj_local[0], ob])]
    sc.obj_mat = [np.concatenate([sc.obj_mat[0], np.ones(n_obj, np.uint32)])]
    return sc


@pytest.mark.parametrize("T", [-1.0, 0.01])
def test_walk_out_of_stack_lockstep(E, T):
    from tests.test_gpu_parity import _lockstep
    _lockstep(E, _crowded(120, 60), 3, T, "crowded box T=%g" % T)


def test_walk_out_of_stack_visibility(E):
    # a point light's visibility tasks walk the whole scene during verification
    from tests.test_gpu_parity import _lockstep
    sc = _crowded(120, 60)
    sc.light_half = np.zeros((1, 2), np.float32)
    sc.light_xforms = sc.light_xforms.copy()
    sc.light_xforms[:, 0, 3] += 0.01 * np.arange(sc.light_xforms.shape[0], dtype=np.float32)
    _lockstep(E, sc, 3, 0.01, "crowded box, moving point light")


def test_ties_between_coincident_triangles(E):
    # every static triangle twice: each closest crossing is a tie, and the
    # paths are those of the scene without the copies, bit for bit
    one = scenes.make_rooms("ties", 2, 2, 3000, 2, (16, 8), 4000 + 5, 5, 3, 0.01, 31, n_lights=2, lights_move=True)
    two = scenes.make_rooms("ties", 2, 2, 3000, 2, (16, 8), 4000 + 5, 5, 3, 0.01, 31, n_lights=2, lights_move=True)
    S = one.n_static
    two.static_verts = np.concatenate([one.static_verts, one.static_verts])
    two.static_mat = np.concatenate([one.static_mat, one.static_mat])
    got = []
    for sc in (one, two):
        ctx = E.Context(sc)
        st = ctx.new_store()
        ctx.frame_begin(0)
        ctx.initial_trace(st, sc.seed, 0)
        for f in (1, 2):
            ctx.frame_begin(f)
            ctx.verify(st)
            ctx.retrace(st, 0.01, sc.seed, f)
        got.append(st.to_numpy())
        ctx.close()
    a, b = got
    for k in ("pos", "energy", "origin"):
        assert np.array_equal(a[k].view(np.uint32), b[k].view(np.uint32)), k
    assert np.array_equal(a["info"], b["info"])
    none = b["hit"] == 0xFFFFFFFF
    hit = np.where(none, b["hit"], np.where(b["hit"] < 2 * S, b["hit"] % S, b["hit"] - S))
    assert np.array_equal(a["hit"], hit)


# Queue, its order, statistics and compaction: a lone path, one below and above
# a chunk of 1,024 paths, and both sides of the sizes from which each list's
# offsets come from a scan of their own (1,048,576 paths for the queue,
# 1,572,864 photon rows for the compaction, 4,194,304 paths for the tasks).
@pytest.mark.parametrize("n,B", [(1, 1), (1023, 3), (1025, 3), (786_433, 2), (1_048_576, 1), (1_048_577, 2),
                                 (1_572_864, 1), (1_572_865, 1), (4_194_304, 1), (4_194_305, 1)])
def test_queue_and_compaction_at_edges(E, n, B):
    import oracle as O
    import torch
    sc = scenes.make_tiny(n_paths=n, max_bounces=B, frames=2, seed=11)
    ctx = E.Context(sc)
    st = ctx.new_store()
    ctx.frame_begin(0)
    ctx.initial_trace(st, 11)
    ctx.frame_begin(1)
    stats = ctx.new_stats()
    ctx.verify(st, stats)
    info = st.info[:n].cpu().numpy().view(np.uint32)
    f = O.info_fields(info)
    queued = f["replace"] != 0
    np.testing.assert_array_equal(ctx.queue(), np.nonzero(queued)[0])
    s = ctx.stats_dict(stats)
    kept = queued & (f["reuse"] != 0)  # replaced from a segment on, the light sample kept
    assert s["paths_invalid"] == queued.sum() and s["paths_light_lost"] == (queued & ~kept).sum()
    assert s["segments_examined"] == f["nseg"][~queued].sum() + (f["start"][kept] + 1).sum()
    # every queued path is re-traced: the rows from its first invalid segment
    # on are overwritten or end before it
    row = torch.arange(B, device="cuda")[:, None]
    q = torch.from_numpy(queued).cuda()
    st.pos_hit[:, :n, :3] = torch.where(
        (q & (row >= torch.from_numpy(f["start"].astype(np.int64)).cuda()))[..., None],
        torch.full((), 1e9, device="cuda"), st.pos_hit[:, :n, :3])
    ctx.retrace(st, -1.0, 11, 1)
    d = st.to_numpy()
    nseg = O.info_fields(d["info"])["nseg"]
    at = np.minimum(f["start"], B - 1)
    left = queued & (nseg > f["start"]) & (d["pos"][at, np.arange(n), 0] == 1e9)
    assert not left.any(), np.nonzero(left)[0][:5]
    np.testing.assert_array_equal(nseg[~queued], f["nseg"][~queued])
    pos, en, cnt = ctx.compact_photons(st)
    there = nseg[None, :] > np.arange(B)[:, None]
    assert cnt == there.sum()
    np.testing.assert_array_equal(pos.cpu().numpy(), d["pos"][there])
    np.testing.assert_array_equal(en.cpu().numpy(), d["energy"][there])
    ctx.close()


# Frame beginning: objects of one triangle, one below and above a 256-record
# block, and both sides of the object size (16,384 triangles) from which boxes
# need the upper pyramid levels; some objects stay where they are in a frame.
@pytest.mark.parametrize("sizes", [[1], [255, 1, 257], [16_384, 2], [16_385, 3, 300]])
def test_object_boxes_at_edges(E, sizes):
    from tests.test_gpu_parity import _lockstep
    sc = scenes.make_tiny(n_paths=1500 + 3, max_bounces=3, frames=4, seed=23)
    rng = np.random.default_rng(len(sizes))
    n_obj = len(sizes)
    sc.obj_local = [(rng.uniform(-0.1, 0.1, (n, 1, 3)) + rng.uniform(-0.02, 0.02, (n, 3, 3))).astype(np.float32)
                    for n in sizes]
    sc.obj_mat = [np.ones(n, np.uint32) for n in sizes]
    base = sc.obj_xforms[:, :1]
    xf = np.repeat(base, n_obj, axis=1).copy()
    for o in range(n_obj):
        xf[:, o, 3] += 0.15 * (o - 1)
    xf[2, 0] = xf[1, 0]  # the first object rests in frame 2
    sc.obj_xforms = xf.astype(np.float32)
    ctx = E.Context(sc)
    for f in range(4):
        ctx.frame_begin(f)
        for o in range(n_obj):
            h = ctx.object_hierarchy_info(o)
            assert h["valid"] and not h["rebuilt"], (f, o, h)
    ctx.close()
    _lockstep(E, sc, 4, 0.01, "objects of %s triangles" % sizes)


# Nodes have origins in scenes of up to 2^20 - 1 triangles: both sides of that
# size, with refit and rebuilt objects, and both kinds in one batch, give the
# paths of the scene without the triangles that nothing can reach.
def _tiny_beside(n_extra):
    sc = scenes.make_tiny(n_paths=1500 + 3, max_bounces=3, frames=4, seed=29)
    rng = np.random.default_rng(29)
    far = (rng.uniform(3.0, 3.2, (n_extra, 1, 3)) + rng.uniform(-1e-3, 1e-3, (n_extra, 3, 3))).astype(np.float32)
    sc.static_verts = np.concatenate([sc.static_verts, far])
    sc.static_mat = np.concatenate([sc.static_mat, np.zeros(n_extra, np.uint32)])
    # the far triangles' side of the box is closed
    wall = np.array([[[0, 0, 1], [1, 1, 1], [0, 1, 1]], [[0, 0, 1], [1, 0, 1], [1, 1, 1]]], np.float32)
    sc.static_verts[:2], keep = wall, sc.static_verts[:2].copy()
    sc.static_verts = np.concatenate([sc.static_verts, keep])
    sc.static_mat = np.concatenate([sc.static_mat, np.zeros(2, np.uint32)])
    return sc


def _three_frames(E, sc):
    ctx = E.Context(sc)
    st = ctx.new_store()
    ctx.frame_begin(0)
    ctx.initial_trace(st, 29)
    out = []
    for f in range(1, 4):
        ctx.set_tuning(object_rebuild=1 if f == 3 else 0)
        ctx.frame_begin(f)
        ctx.verify(st)
        ctx.retrace(st, 0.01, 29, f)
        d = st.to_numpy()
        out.append({k: d[k] for k in ("pos", "energy", "info", "origin")})
    ctx.close()
    return out


def test_scene_sizes_with_and_without_node_origins(E):
    plain = _three_frames(E, _tiny_beside(0))
    n = (1 << 20) - 1 - (12 + 12)  # box and cube: 24 triangles
    for extra in (n, n + 1):
        for f, (a, b) in enumerate(zip(plain, _three_frames(E, _tiny_beside(extra)))):
            for k in a:
                np.testing.assert_array_equal(a[k], b[k], err_msg="%s, frame %d, %d extra" % (k, f + 1, extra))
    scs = [_tiny_beside(0), _tiny_beside(n + 1)]
    ctxs = [E.Context(sc) for sc in scs]
    sts = [c.new_store() for c in ctxs]
    for c, st in zip(ctxs, sts):
        c.frame_begin(0)
        c.initial_trace(st, 29)
    bt = E.Batch(ctxs, sts, 0.01, 29)
    for f in (1, 2):
        bt.frame(f)
        for st in sts:
            d = st.to_numpy()
            for k in plain[f - 1]:
                np.testing.assert_array_equal(plain[f - 1][k], d[k], err_msg="batch %s, frame %d" % (k, f))
    bt.close()
    for c in ctxs:
        c.close()


# The rebuild's sort: one triangle, both sides of a wave, of a round of 1,024,
# of the two sizes (8,192 and 16,384 triangles) that one workgroup sorts, with
# many equal codes.  The hierarchies are those of the sort in passes, which an
# object past that size brings for all of them.
@pytest.mark.parametrize("n", [2, 64, 65, 1024, 1025, 8192, 8193, 16_383, 16_384])
def test_small_and_large_sorts_agree(E, n):
    def objects(more):
        rng = np.random.default_rng(n)
        tris = (rng.integers(-20, 21, (n, 1, 3)) * 0.005 + rng.uniform(-0.02, 0.02, (1, 3, 3))).astype(np.float32)
        big = (rng.uniform(-0.05, 0.05, (16385, 1, 3)) + rng.uniform(-0.01, 0.01, (16385, 3, 3))).astype(np.float32)
        sc = scenes.make_tiny(n_paths=1200, max_bounces=3, frames=3, seed=31)
        sc.obj_local = [tris, big[:16385] if more else big[:1], tris[:1]]
        sc.obj_mat = [np.ones(len(t), np.uint32) for t in sc.obj_local]
        xf = np.repeat(sc.obj_xforms, 3, axis=1).copy()
        for o in range(3):
            xf[:, o, 3] += 0.2 * o
        sc.obj_xforms = xf
        return sc

    infos = []
    for more in (0, 1):
        ctx = E.Context(objects(more))
        ctx.set_tuning(object_rebuild=1)
        for f in range(2):
            ctx.frame_begin(f)
        infos.append([ctx.object_hierarchy_info(o) for o in range(3)])
        for o, h in enumerate(infos[-1]):
            assert h["valid"], (o, h)
        ctx.close()
    for o in (0, 2):
        assert infos[0][o] == infos[1][o], (o, infos[0][o], infos[1][o])
