"""The kernel that a call's fused z pass runs, as the library reports it
(Plan.z_form), for every length, channel count and batch that the wave and
register forms take; and the wave form's bits where every row of the spectrum
has a mirror row (directions with a z parity), against the single-group form."""
import pytest

from paper_1804_01830_amd import workloads as W

pytestmark = pytest.mark.gpu

AXES = [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0)]
LINES = [(0.0, 0.0, 1.0), (0.6, 0.0, 0.8), (0.0, 0.6, 0.8)]


def _plan(n, lines, nb, prec, tile=None):
    import torch
    assert torch.cuda.is_available()
    from paper_1804_01830_amd import binding as B
    desc = B.make_desc(n, (1.0, 1.0, 2.0), 1.0, 0.3, lines, precision=prec, batch=nb)
    if tile is None:
        return B.Plan(desc)
    d = B.Plan(desc).info()
    t = B.Tuning()
    t.rows_x, t.tk_y, t.ex, t.ey, t.tk_z, t.ez, t.z_groups = d.rows_x, d.tile_y, d.ex, d.ey, tile, d.ez, 1
    return B.Plan(desc, tuning=t)


# layers, channels / 3, precision, realisations -> kernel
FORMS = [(4, 1, 32, 1, "k_z_wave"), (8, 2, 32, 2, "k_z_wave"), (32, 2, 32, 1, "k_z_wave"), (64, 1, 32, 1, "k_z_wave"),
         (64, 2, 32, 1, "k_z_serial"), (8, 3, 32, 1, "k_z_serial"), (8, 2, 32, 3, "k_z_reg"), (16, 1, 32, 3, "k_z_reg"),
         (32, 1, 32, 12, "k_z_reg"), (32, 2, 32, 4, "k_z_reg"), (64, 2, 32, 4, "k_z_reg"), (64, 3, 32, 4, "k_z_serial"),
         (8, 1, 64, 5, "k_z_wave"), (64, 2, 64, 2, "k_z_wave"), (8, 3, 64, 2, "k_z_serial"), (2, 1, 64, 16, "k_z_grouped")]


@pytest.mark.parametrize("nz,lines,prec,nb,kernel", FORMS)
def test_reported_form(nz, lines, prec, nb, kernel):
    p = _plan((9, 8, nz), LINES[:lines], nb, prec)
    name, tile, threads, blocks = p.z_form()
    print(f"[z form] nz {nz} C {3 * lines} FP{prec} B {nb}: {name} tile {tile} threads {threads} blocks {blocks}",
          flush=True)
    assert name == kernel and tile == p.info().tile_z and threads % 64 == 0 and blocks >= 16
    p.close()


# grid, realisations: every length of the wave form, partial and full layers,
# one and several waves a block
PARITY = [((9, 7, 3), 2), ((5, 9, 7), 1), ((20, 6, 8), 2), ((9, 8, 12), 1), ((5, 7, 16), 2), ((9, 8, 25), 2),
          ((20, 6, 32), 1), ((5, 7, 50), 1), ((9, 5, 64), 2)]


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("n,nb", PARITY)
def test_wave_form_with_mirrored_rows_gives_the_bits_of_the_single_group_form(n, nb, prec):
    import torch
    length = max(2, 1 << (2 * n[2] - 2).bit_length())
    # six channels, unstaged; three at length 128 in FP32, where the wave form does not take six
    lines = AXES[:1] if prec == 32 and length == 128 else AXES
    w = W.random_field(n, lines=lines, batch=nb, seed=83, d=(1.0, 1.0, 2.0))
    dt = torch.float32 if prec == 32 else torch.float64
    rho = torch.from_numpy(w["rho"]).to("cuda", dtype=dt).contiguous()
    outs = []
    for tile, kernel in ((256 // length, "k_z_wave"), (2 if length == 8 else 512 // length, "k_z_serial")):
        p = _plan(n, lines, nb, prec, tile)
        assert p.z_form()[0] == kernel and p.info().mirror_z == 1 and p.info().padded[2] == length
        out = p.new_output()
        p.set_density(rho)
        p.stress(out)
        torch.cuda.synchronize()
        outs.append(out)
        p.close()
    print(f"[z wave form] {n} B={nb} FP{prec} length {length} mirrored", flush=True)
    assert torch.equal(outs[0], outs[1])
