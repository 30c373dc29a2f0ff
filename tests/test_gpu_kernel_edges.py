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
