"""The fused x-y kernels on planes up to Py = 128, Px = 256 (both precisions):
the stages and products of the separate passes, so the same bits."""
import pytest

from paper_1804_01830_amd import workloads as W

pytestmark = pytest.mark.gpu

# grid, periodic axes: every column length (16 to 128) and half row length (8
# to 128), the smallest and full number of rows, odd rows (unpaired access),
# rows that fill their waves unevenly, full rows and columns (periodic axes)
CASES = [((5, 5, 3), (False, False)), ((8, 8, 5), (False, False)), ((9, 7, 4), (False, False)),
         ((100, 6, 3), (False, False)), ((33, 8, 2), (False, False)),
         ((7, 9, 3), (False, False)), ((16, 16, 2), (False, False)), ((65, 13, 3), (False, False)),
         ((128, 16, 2), (False, False)), ((20, 17, 3), (False, False)), ((32, 32, 4), (False, False)),
         ((8, 31, 2), (False, False)), ((50, 29, 3), (False, False)), ((127, 30, 2), (False, False)),
         ((6, 33, 2), (False, False)), ((16, 64, 2), (False, False)), ((31, 50, 3), (False, False)),
         ((64, 64, 2), (False, False)), ((101, 63, 2), (False, False)),
         ((16, 16, 3), (True, True)), ((256, 16, 2), (True, True)), ((9, 32, 2), (False, True)),
         ((64, 20, 2), (True, False)), ((64, 64, 3), (True, True)), ((128, 128, 2), (True, True))]


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("n,periodic", CASES)
def test_fused_planes_give_the_bits_of_the_separate_passes(n, periodic, prec):
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_field(n, n_lines=1, batch=2, seed=61, d=(1.0, 1.0, 2.0))
    desc = B.make_desc(w["n"], w["d"], w["mu"], w["nu"], w["lines"], precision=prec, batch=2, periodic=periodic,
                       pbc_shells=2)
    plan = B.Plan(desc)
    i = plan.info()
    assert i.xy_fused == 1 and i.yx_fused == 1
    t = B.Tuning()
    t.rows_x, t.tk_y, t.ex, t.ey, t.tk_z, t.ez, t.z_groups = (i.rows_x, i.tile_y, i.ex, i.ey, i.tile_z, i.ez,
                                                              i.z_groups)
    t.yx = t.xy = 1
    other = B.Plan(desc, tuning=t)
    assert other.info().xy_fused == 0 and other.info().yx_fused == 0
    dt = torch.float32 if prec == 32 else torch.float64
    rho = torch.from_numpy(w["rho"]).to("cuda", dtype=dt).contiguous()
    outs, stats = [], []
    for p in (plan, other):
        out = p.new_output()
        st = torch.zeros((2, 6, n[2]), dtype=torch.float64, device="cuda")
        p.set_plane_stats(st)
        p.set_density(rho)
        p.stress(out)
        torch.cuda.synchronize()
        outs.append(out)
        stats.append(st)
    print(f"[fused planes] {n} {periodic} FP{prec} padded {tuple(i.padded)}", flush=True)
    assert torch.equal(outs[0], outs[1])
    # sums of at most 2^14 squares in double, in another order: 2^14 x 2^-53 relative
    assert torch.allclose(stats[0], stats[1], rtol=2e-12, atol=0)
    plan.close()
    other.close()


@pytest.mark.parametrize("n", [(64, 64, 16), (20, 64, 16)])
def test_many_double_planes_give_the_same_bits_every_time(n):
    """Planes that share CUs (768 of them), whose wide stores have to wait."""
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_field(n, n_lines=1, batch=16, seed=62, d=(1.0, 1.0, 2.0))
    desc = B.make_desc(w["n"], w["d"], w["mu"], w["nu"], w["lines"], precision=64, batch=16)
    plan = B.Plan(desc)
    i = plan.info()
    t = B.Tuning()
    t.rows_x, t.tk_y, t.ex, t.ey, t.tk_z, t.ez, t.z_groups = (i.rows_x, i.tile_y, i.ex, i.ey, i.tile_z, i.ez,
                                                              i.z_groups)
    t.yx = t.xy = 1
    other = B.Plan(desc, tuning=t)
    rho = torch.from_numpy(w["rho"]).to("cuda").contiguous()
    ref, out = other.new_output(), plan.new_output()
    other.set_density(rho)
    other.stress(ref)
    print(f"[fused planes] {n} FP64, 16 realisations, 20 evaluations", flush=True)
    for _ in range(20):
        plan.set_density(rho)
        plan.stress(out)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    plan.close()
    other.close()
