"""The hierarchies that the kernels walk, as the device wrote them: planes,
origins, units and child codes of the four-wide form, and the order that the
rebuild's sorts give, by the library's own check (binary and four-wide form,
every triangle in one leaf, inside every box on the way, leaves in the stable
order of their codes)."""
import numpy as np
import pytest

from paper_2111_06906_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_2111_06906_amd import engine
    return engine


def _scene(sizes, seed, static_extra=0, far=0.0, n_paths=1200):
    rng = np.random.default_rng(seed)
    sc = scenes.make_tiny(n_paths=n_paths, max_bounces=3, frames=4, seed=31)
    # few distinct centroids, so that many codes are equal, and scattered ones
    sc.obj_local = [np.concatenate([
        (rng.integers(-20, 21, (n // 2, 1, 3)) * 0.004 + rng.uniform(-0.02, 0.02, (1, 3, 3))),
        (rng.uniform(-0.08, 0.08, (n - n // 2, 1, 3)) + rng.uniform(-0.01, 0.01, (n - n // 2, 3, 3)))]).astype(np.float32)
        for n in sizes]
    sc.obj_mat = [np.ones(n, np.uint32) for n in sizes]
    xf = np.repeat(sc.obj_xforms[:, :1], len(sizes), axis=1).copy()
    for o in range(len(sizes)):
        xf[:, o, 3] += 0.15 * (o - 1)
    xf[2, 0] = xf[1, 0]  # the first object rests in frame 2
    xf[1:3, -1, 7] += far  # the last one leaves and returns
    sc.obj_xforms = xf.astype(np.float32)
    if static_extra:
        t = (rng.uniform(3.0, 3.2, (static_extra, 1, 3)) + rng.uniform(-1e-3, 1e-3, (static_extra, 3, 3))).astype(np.float32)
        sc.static_verts = np.concatenate([sc.static_verts, t])
        sc.static_mat = np.concatenate([sc.static_mat, np.zeros(static_extra, np.uint32)])
    return sc


def _check(E, sc, rebuild, frames=4):
    ctx = E.Context(sc)
    ctx.set_tuning(object_rebuild=rebuild)
    for f in range(frames):
        ctx.frame_begin(f)
        for o, t in enumerate(sc.obj_local):
            h = ctx.object_hierarchy_info(o)
            assert h["valid"] and h["rebuilt"] == bool(rebuild and len(t) > 1), (f, o, len(t), h)
            if rebuild:
                assert h["leaves"] == len(t), (f, o, h)
    ctx.close()


# Objects of one triangle, both sides of a wave, of a round of the sort, of the
# two sizes that one workgroup sorts, and past them: the passes' order is checked
# against the same stable order.
@pytest.mark.parametrize("rebuild", [0, 1])
@pytest.mark.parametrize("sizes", [[1, 2, 3], [64, 65, 1], [1024, 1025], [8192, 5], [8193, 300], [16_384, 8], [16_385, 64],
                                   [40_000, 2, 1025]])
def test_written_hierarchies(E, sizes, rebuild):
    _check(E, _scene(sizes, sum(sizes)), rebuild)


# Objects that bring units of their own (40 to 10^7 units away) and scenes too
# large for origins.
@pytest.mark.parametrize("rebuild", [0, 1])
@pytest.mark.parametrize("extra,far", [(0, 40.0), (0, -3000.0), (0, 1e7), ((1 << 20), 0.0), ((1 << 20), 1e5)])
def test_written_hierarchies_with_units_and_without_origins(E, extra, far, rebuild):
    _check(E, _scene([300, 65, 1025], 7, extra, far), rebuild)


@pytest.mark.parametrize("n", [8192, 8193, 16_384, 16_385])
def test_rebuilt_objects_lockstep_at_sort_sizes(E, n):
    from tests.test_gpu_parity import _lockstep
    _lockstep(E, _scene([n, 300], n, n_paths=1503), 3, 0.01, "rebuilt object of %d triangles" % n,
              tuning=dict(object_rebuild=1))
