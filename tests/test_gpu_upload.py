"""Uploads into one context in turn: small arrays share a block and a copy, larger
ones have their own, at both sides of either size; every scene traces as in a
context of its own."""
import numpy as np
import pytest

from paper_2111_06906_amd import scenes

pytestmark = pytest.mark.gpu


def _scene(n_static, n_obj, seed):
    sc = scenes.make_tiny(n_paths=1200, max_bounces=3, frames=3, seed=seed)
    rng = np.random.default_rng(seed)
    extra = (rng.uniform(0.1, 0.9, (n_static, 1, 3)) + rng.uniform(-0.02, 0.02, (n_static, 3, 3))).astype(np.float32)
    sc.static_verts = np.concatenate([sc.static_verts, extra])
    sc.static_mat = np.concatenate([sc.static_mat, np.zeros(n_static, np.uint32)])
    obj = (rng.uniform(-0.08, 0.08, (n_obj, 1, 3)) + rng.uniform(-0.01, 0.01, (n_obj, 3, 3))).astype(np.float32)
    sc.obj_local = [np.concatenate([sc.obj_local[0], obj])]
    sc.obj_mat = [np.concatenate([sc.obj_mat[0], np.ones(n_obj, np.uint32)])]
    return sc


def _trace(ctx):
    st = ctx.new_store()
    ctx.frame_begin(0)
    ctx.initial_trace(st, 3)
    for f in (1, 2):
        ctx.frame_begin(f)
        ctx.verify(st)
        ctx.retrace(st, 0.01, 3, f)
    assert ctx.object_hierarchy_info(0)["valid"]
    return st.to_numpy()


def test_uploads_in_turn_match_fresh_contexts():
    from paper_2111_06906_amd import _lib as L
    from paper_2111_06906_amd import engine
    # records: 64 bytes each, 64 KiB at 1,024; ids: 4 bytes, 64 KiB at 16,384; many
    # small arrays past one block at 10,000
    sizes = [(0, 0), (1000, 0), (1001, 1), (1002, 10), (40_000, 20), (0, 2000), (16_300, 60), (16_390, 60), (10_000, 6000),
             (3, 0)]
    ctx = None
    for seed, (a, b) in enumerate(sizes):
        sc = _scene(a, b, seed)
        if ctx is None:
            ctx = engine.Context(sc)
        else:
            ctx.scene = sc
            ctx._upload(sc)
            counts = np.ascontiguousarray(sc.light_paths, np.uint32)
            L.set_light_paths(ctx.ctx, engine._np_ptr(counts))
        fresh = engine.Context(sc)
        x, y = _trace(ctx), _trace(fresh)
        fresh.close()
        for k in x:
            np.testing.assert_array_equal(x[k], y[k], err_msg="%s of %s" % (k, (a, b)))
    ctx.close()
