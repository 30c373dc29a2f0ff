"""Gradients where an accumulator takes its largest number of additions."""
import numpy as np
import pytest

from paper_2111_06906_amd import scenes

pytestmark = pytest.mark.gpu


# 256 materials, of which one takes 95% of the hits, at 15 bounces: accumulators
# shared by eight lanes, up to 112 additions a round to one of them.  At most 224
# roundings of random sign in a partial sum come to about 7.5 x 2^-24 of it, those
# of the terms (under 50 x 2^-24 each, independent) and of thousands of partial
# sums average out, and the result rounds once: 8 x 2^-24.
@pytest.mark.parametrize("n,n_mat,B,seed", [(1_600_003, 256, 15, 6), (400_003, 120, 15, 2),
                                            (1_000_003, 60, 7, 3)])
def test_one_material_takes_nearly_all_hits(n, n_mat, B, seed):
    import torch
    from paper_2111_06906_amd import engine
    g = torch.Generator(device="cuda").manual_seed(seed)

    def uniform(*shape, lo=0.0, hi=1.0):
        return lo + (hi - lo) * torch.rand(shape, generator=g, device="cuda")

    T, L = 5000, 2
    mat = torch.where(uniform(T) < 0.95, 0, torch.randint(0, n_mat, (T,), generator=g, device="cuda"))
    hit = torch.randint(0, T, (B, n), generator=g, device="cuda", dtype=torch.int32)
    nseg = torch.where(uniform(n) < 0.1, torch.randint(0, B + 1, (n,), generator=g, device="cuda"), B)
    albedo, power, gE = uniform(n_mat, 3, lo=0.3, hi=0.8), uniform(L, 3, lo=0.5, hi=2.0), uniform(B, n, 3)
    counts = np.array([n - n // 2, n // 2], np.int64)
    tri = np.random.default_rng(seed).uniform(-1, 1, (T, 3, 3)).astype(np.float32)
    sc = scenes.Scene(
        name="one material", static_verts=tri, static_mat=mat.cpu().numpy().astype(np.uint32), obj_local=[], obj_mat=[],
        obj_xforms=np.zeros((1, 0, 12), np.float32), albedo=albedo.cpu().numpy(),
        light_half=np.full((L, 2), 0.05, np.float32), light_power=power.cpu().numpy(),
        light_xforms=np.tile(np.array([1, 0, 0, 0, 0, 0, -1, 0.9, 0, 1, 0, 0], np.float32), (1, L, 1)),
        light_paths=counts, max_bounces=B, threshold=0.01, seed=1)
    ctx = engine.Context(sc)
    st = ctx.new_store()
    st.pos_hit.view(torch.int32)[:, :n, 3] = hit
    st.info[:n] = nseg.to(torch.int32) << 22
    ga, gp = ctx.energy_backward(st, albedo, power, gE)
    rho, phi = albedo.double().requires_grad_(True), power.double().requires_grad_(True)
    light = torch.repeat_interleave(torch.arange(L, device="cuda"), torch.as_tensor(counts, device="cuda"))
    e = phi[light] / torch.as_tensor(counts, device="cuda")[light].double()[:, None]
    total = 0.0
    for r in range(B):
        if r:
            e = e * rho[mat[hit[r - 1].long()]]
        total = total + (e * (nseg > r)[:, None] * gE[r].double()).sum()
    total.backward()
    for got, ref in ((ga[:1], rho.grad[:1]), (gp, phi.grad)):
        err = ((got.double() - ref).abs() / ref).max().item()
        assert err <= 8 * 2.0 ** -24, err
    ctx.close()
