"""Element classes left at 0 in a tuning are those of the default plan."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("n", [(9, 16, 4), (9, 70, 3), (9, 128, 4), (9, 150, 3)])
def test_zero_selects_the_default_classes(n, precision):
    import torch
    from paper_1804_01830_amd import binding as B
    assert torch.cuda.is_available()
    desc = B.make_desc(n, (1.0, 1.0, 2.0), 1.0, 0.3, [(0.0, 0.0, 1.0)], precision=precision)
    plan = B.Plan(desc)
    i = plan.info()
    t = B.Tuning()
    t.rows_x, t.tk_y, t.tk_z = i.rows_x, i.tile_y, i.tile_z
    tuned = B.Plan(desc, tuning=t)
    u = tuned.info()
    print(f"[tuning defaults] {n} FP{precision} classes {u.ex} {u.ey} {u.ez}", flush=True)
    assert (u.ex, u.ey, u.ez, u.z_groups, u.xy_fused, u.yx_fused) == \
        (i.ex, i.ey, i.ez, i.z_groups, i.xy_fused, i.yx_fused)
    tuned.close()
    plan.close()
