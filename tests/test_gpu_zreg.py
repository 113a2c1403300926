"""The register form of the fused z pass (FP32, z lengths 16 to 128, plans of
several realisations): its arithmetic is that of the single-group form, so the
two agree bit for bit. The form is chosen by tile width, so a plan forced to
another tile runs the single-group form; calls on few realisations of the same
plan run the single-group form too."""
import pytest

from paper_1804_01830_amd import workloads as W

pytestmark = pytest.mark.gpu

AXES = [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0)]

# grid, line directions (a count, or directions with a z parity), realisations:
# every z length at its smallest, a partial and the full number of layers; x
# lengths that end in a Nyquist strip (9, 20) and in a shared last tile (5, 40);
# batches that fill the waves of a block unevenly
CASES = [
    ((9, 7, 5), 2, 3), ((20, 6, 8), 3, 5), ((5, 9, 7), AXES[:2], 4),
    ((9, 5, 9), 1, 3), ((20, 7, 16), 2, 6), ((40, 6, 12), 3, 4), ((9, 6, 11), AXES, 9),
    ((9, 5, 17), 1, 13), ((20, 7, 32), 1, 16), ((40, 6, 25), 2, 4), ((9, 8, 32), 3, 5), ((20, 5, 20), AXES, 4),
    ((9, 5, 33), 1, 4), ((20, 6, 64), 2, 5), ((5, 7, 50), AXES[:2], 6),
]


@pytest.mark.parametrize("n,lines,nb", CASES)
def test_register_form_gives_the_bits_of_the_single_group_form(n, lines, nb):
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_field(n, batch=nb, seed=51, d=(1.0, 1.0, 2.0),
                       **(dict(n_lines=lines) if isinstance(lines, int) else dict(lines=lines)))
    desc = B.make_desc(w["n"], w["d"], w["mu"], w["nu"], w["lines"], precision=32, batch=nb)
    plan = B.Plan(desc)
    i = plan.info()
    assert i.z_groups == 1 and i.ez == 4 and i.tile_z == (8 if i.padded[2] == 128 else 16)
    t = B.Tuning()
    t.rows_x, t.tk_y, t.ex, t.ey, t.tk_z, t.ez, t.z_groups = i.rows_x, i.tile_y, i.ex, i.ey, 4, 4, 1
    other = B.Plan(desc, tuning=t)
    rho = torch.from_numpy(w["rho"]).to("cuda", dtype=torch.float32).contiguous()
    outs = []
    for p in (plan, other):
        out = p.new_output()
        p.set_density(rho)
        p.stress(out)
        outs.append(out)
    few = torch.empty((2, 6, *rho.shape[2:]), dtype=torch.float32, device="cuda")
    plan.stress_batch(rho[1:3].contiguous(), few, 2)
    torch.cuda.synchronize()
    print(f"[z register form] {n} C={i.channels} B={nb} mirror_z={i.mirror_z}", flush=True)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(few, outs[0][1:3])
    plan.close()
    other.close()
