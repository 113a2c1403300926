"""The wave form of the fused z pass with four elements per thread (z lengths 8
to 128; FP64, and FP32 with one or two realisations): the stages and sums of
the single-group form, so the same bits. The form is chosen by tile width, so a
plan forced to another tile runs the single-group form."""
import pytest

from paper_1804_01830_amd import workloads as W

pytestmark = pytest.mark.gpu

AXES = [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0)]

# grid, line directions (a count, or directions with a z parity), realisations:
# every z length at its smallest, a partial and the full number of layers; x
# lengths that end in a Nyquist strip or in a shared last tile; batches that
# fill the waves of a block unevenly
CASES = [((9, 7, 3), 1, 2), ((20, 6, 4), 2, 3), ((9, 7, 5), 2, 1), ((20, 6, 8), 1, 2), ((5, 9, 7), AXES, 5),
         ((9, 5, 9), 1, 1), ((20, 7, 16), 2, 2), ((40, 6, 12), 1, 6), ((9, 5, 17), 2, 2), ((20, 7, 32), 1, 1),
         ((40, 6, 25), 1, 5), ((9, 8, 32), AXES, 2), ((9, 5, 33), 1, 2), ((20, 6, 64), 2, 1), ((5, 7, 50), AXES, 3)]


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("n,lines,nb", CASES)
def test_wave_form_gives_the_bits_of_the_single_group_form(n, lines, nb, prec):
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_field(n, batch=nb, seed=81, d=(1.0, 1.0, 2.0),
                       **(dict(n_lines=lines) if isinstance(lines, int) else dict(lines=lines)))
    desc = B.make_desc(w["n"], w["d"], w["mu"], w["nu"], w["lines"], precision=prec, batch=nb)
    d = B.Plan(desc).info()
    P = d.padded[2]
    dt = torch.float32 if prec == 32 else torch.float64
    rho = torch.from_numpy(w["rho"]).to("cuda", dtype=dt).contiguous()
    outs, few = [], []
    for tile in (256 // P, 2 if P == 8 else 512 // P):
        t = B.Tuning()
        t.rows_x, t.tk_y, t.ex, t.ey, t.tk_z, t.z_groups = d.rows_x, d.tile_y, d.ex, d.ey, tile, 1
        t.ez = 4 if prec == 32 else 2
        p = B.Plan(desc, tuning=t)
        out = p.new_output()
        p.set_density(rho)
        p.stress(out)
        one = torch.empty((1, 6, *rho.shape[2:]), dtype=dt, device="cuda")
        p.stress_batch(rho[nb - 1:].contiguous(), one, 1)
        torch.cuda.synchronize()
        outs.append(out)
        few.append(one)
        p.close()
    print(f"[z wave form] {n} C={d.channels} B={nb} FP{prec} length {P} mirror_z={d.mirror_z}", flush=True)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(few[0], few[1]) and torch.equal(few[0][0], outs[0][nb - 1])
