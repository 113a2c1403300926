"""A plan that shares the spectrum of a plan of fewer realisations runs the z
kernel and the tile of its own calls, whose blocks then read several of the
spectrum's narrower tiles: the same kernel as a plan built for that batch, and
the same bits."""
import pytest

from paper_1804_01830_amd import workloads as W

pytestmark = pytest.mark.gpu

AXES = [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0)]

# grid, line directions (a count, or directions with a z parity), realisations of
# the source and of the shared plan: z lengths 16 to 128; x lengths whose last block
# ends inside the spectrum's tiles (9, 20, 40) and whose plane is narrower than a
# block (5); sources without and with a Nyquist strip
CASES = [((9, 7, 8), 2, 1, 4), ((20, 8, 12), 2, 1, 3), ((20, 6, 16), 1, 1, 4), ((40, 8, 9), 3, 1, 5),
         ((9, 8, 16), AXES, 1, 3), ((5, 9, 12), 2, 1, 4), ((9, 8, 32), 1, 1, 13), ((40, 6, 20), 1, 1, 4),
         ((20, 9, 32), 2, 1, 5), ((5, 6, 25), 3, 1, 4), ((9, 8, 30), AXES[:2], 1, 6), ((9, 8, 64), 1, 1, 4),
         ((40, 64, 32), [(0.6, 0.0, 0.8)], 1, 7), ((30, 40, 50), 1, 1, 3), ((9, 8, 50), 1, 1, 3), ((20, 6, 50), 2, 1, 5), ((40, 7, 64), 1, 1, 6), ((5, 8, 33), 1, 1, 4), ((9, 8, 64), AXES[:2], 1, 4),
         ((40, 12, 32), 1, 4, 13), ((20, 30, 32), 1, 5, 12), ((5, 9, 32), 1, 4, 12)]


@pytest.mark.parametrize("n,lines,src,nb", CASES)
def test_shared_plans_run_the_form_of_their_batch(n, lines, src, nb):
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_field(n, batch=nb, seed=91, d=(1.0, 1.0, 2.0),
                       **(dict(n_lines=lines) if isinstance(lines, int) else dict(lines=lines)))
    desc = B.make_desc(w["n"], w["d"], w["mu"], w["nu"], w["lines"], precision=32, batch=nb)
    direct = B.Plan(desc)
    desc.batch = src
    shared = B.Plan(desc).share(nb)
    rho = torch.from_numpy(w["rho"]).to("cuda", dtype=torch.float32).contiguous()
    ref, out = direct.new_output(), torch.empty_like(direct.new_output())
    direct.stress_batch(rho, ref, nb)
    for k in sorted({1, 2, 3, nb}):
        if k > nb:
            continue
        out.fill_(float("nan"))
        shared.stress_batch(rho[:k].contiguous(), out[:k], k)
        torch.cuda.synchronize()
        print(f"[shared form] {n} C={direct.channels} from {src}, {k} of {nb}: {shared.z_form(k)[:2]} on tile "
              f"{shared.info().tile_z}, direct {direct.z_form()[:2]}", flush=True)
        assert torch.equal(out[:k], ref[:k])
    if n[0] == 5 and src > 1:        # the strip of the source's tile is none of a wider block's: kept
        assert shared.z_form()[:2] == ("k_z_serial", shared.info().tile_z)
    elif nb == 7:                    # 16 columns without a z parity do not fit the LDS: eight
        assert shared.z_form()[:2] == ("k_z_serial", 8)
    elif n in ((9, 8, 50), (40, 6, 20)):    # too small a call for wider tiles of the single-group form
        assert shared.z_form()[:2] == ("k_z_serial", shared.info().tile_z)
    else:
        assert shared.z_form()[:2] == direct.z_form()[:2]
    shared.close()
    direct.close()


@pytest.mark.parametrize("n,lines", [((9, 8, 32), 2), ((20, 8, 64), 1), ((20, 8, 16), 1)])
def test_a_tuning_holds_for_its_batch(n, lines):
    """Sharers of a tuned plan run its tile up to its batch, and the form of their own beyond."""
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_field(n, batch=4, seed=92, d=(1.0, 1.0, 2.0), n_lines=lines)
    desc = B.make_desc(w["n"], w["d"], w["mu"], w["nu"], w["lines"], precision=32, batch=4)
    direct = B.Plan(desc)
    desc.batch = 1
    i = B.Plan(desc).info()
    t = B.Tuning()
    t.rows_x, t.tk_y, t.ex, t.ey, t.tk_z, t.ez, t.z_groups = (i.rows_x, i.tile_y, i.ex, i.ey, i.tile_z, i.ez, 1)
    tuned = B.Plan(desc, tuning=t)
    shared = tuned.share(4)
    assert shared.z_form(1)[:2] == tuned.z_form()[:2] and tuned.z_form()[1] == t.tk_z
    assert shared.z_form(4)[:2] == direct.z_form()[:2] and shared.info().tile_z == t.tk_z
    rho = torch.from_numpy(w["rho"]).to("cuda", dtype=torch.float32).contiguous()
    ref, out = direct.new_output(), direct.new_output()
    direct.stress_batch(rho, ref, 4)
    shared.stress_batch(rho, out, 4)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    for p in (shared, tuned, direct):
        p.close()
