"""The fused x-y kernels against the separate passes on both sides of the number
of planes from which a call takes them: the same bits from calls on few and on
many realisations, and each call on the path that the count selects."""
import pytest

from paper_1804_01830_amd import workloads as W

pytestmark = pytest.mark.gpu

# grid, periodic axes, precision, realisations, fused forward, fused inverse (three
# channels: 3 B Nz planes forward, 6 B Nz inverse)
CASES = [((16, 50, 5), False, 64, 5, True, False), ((16, 50, 6), False, 64, 5, True, True),
         ((30, 64, 3), False, 64, 6, True, False), ((32, 64, 5), False, 64, 4, True, True),
         ((50, 33, 5), False, 64, 2, True, False), ((64, 64, 3), False, 64, 4, True, True),
         ((100, 64, 5), False, 64, 2, False, False), ((128, 40, 4), False, 64, 4, True, True),
         ((16, 128, 4), True, 64, 1, True, True), ((32, 128, 4), True, 64, 2, False, False),
         ((32, 128, 9), True, 64, 3, True, True), ((64, 128, 6), True, 64, 2, False, False),
         ((64, 128, 11), True, 64, 2, True, True), ((128, 128, 7), True, 64, 3, False, True),
         ((128, 128, 11), True, 64, 2, True, True), ((256, 64, 5), True, 64, 1, False, True),
         ((256, 64, 3), True, 64, 2, True, True), ((32, 128, 4), True, 32, 4, False, False),
         ((32, 128, 11), True, 32, 2, True, True), ((64, 128, 13), True, 32, 1, False, False),
         ((64, 128, 7), True, 32, 2, False, True), ((128, 128, 5), True, 32, 2, False, False),
         ((128, 128, 22), True, 32, 1, True, True), ((256, 128, 5), True, 32, 1, False, False),
         ((256, 128, 3), True, 32, 2, False, True), ((64, 64, 1), False, 32, 1, True, True)]


@pytest.mark.parametrize("n,periodic,prec,nb,forward,inverse", CASES)
def test_both_paths_give_the_same_bits(n, periodic, prec, nb, forward, inverse):
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_field(n, n_lines=1, batch=nb, seed=71, d=(1.0, 1.0, 2.0))
    desc = B.make_desc(w["n"], w["d"], w["mu"], w["nu"], w["lines"], precision=prec, batch=nb,
                       periodic=(periodic, periodic), pbc_shells=1)
    plan = B.Plan(desc)
    i = plan.info()
    assert i.xy_fused == 1 and i.yx_fused == 1
    t = B.Tuning()
    t.rows_x, t.tk_y, t.ex, t.ey, t.tk_z, t.ez, t.z_groups = (i.rows_x, i.tile_y, i.ex, i.ey, i.tile_z, i.ez,
                                                              i.z_groups)
    t.yx = t.xy = 1
    other = B.Plan(desc, tuning=t)
    dt = torch.float32 if prec == 32 else torch.float64
    rho = torch.from_numpy(w["rho"]).to("cuda", dtype=dt).contiguous()
    out, ref = plan.new_output(), other.new_output()
    plan.set_density(rho)
    other.set_density(rho)
    passes = plan.time_passes(out, 1)
    separate = other.time_passes(ref, 1)
    one = torch.empty((1, *out.shape[1:]), dtype=dt, device="cuda")
    stats, sref = (torch.zeros((nb, 6, n[2]), dtype=torch.float64, device="cuda") for _ in range(2))
    plan.stress_batch(rho[nb - 1:].contiguous(), one, 1)
    out.zero_()
    plan.stress_batch_stats_noalloc(rho, out, nb, stats)
    other.stress_batch_stats_noalloc(rho, ref, nb, sref)
    torch.cuda.synchronize()
    print(f"[plane count] {n} periodic {periodic} FP{prec} B {nb}: forward fused {passes['y_fwd'] == 0}, inverse fused "
          f"{passes['x_c2r'] == 0}", flush=True)
    assert (passes["y_fwd"] == 0) == forward and (passes["x_c2r"] == 0) == inverse
    assert separate["y_fwd"] > 0 and separate["x_c2r"] > 0
    assert torch.equal(out, ref) and torch.equal(one[0], ref[nb - 1])
    # sums of at most 2^15 squares in double, in another order: 2^15 x 2^-53 relative
    assert torch.allclose(stats, sref, rtol=4e-12, atol=0)
    plan.set_graph(True)
    for _ in range(3):                   # captured once, replayed after
        out.zero_()
        plan.stress_batch(rho, out, nb)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    plan.close()
    other.close()
