"""Steps taken one call at a time, each starting from ghost layers that are
there, against the same steps in one call, which forms them on the way: the
same bits, ghost layers included."""
import pytest

from paper_1804_01830_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("n", [(64, 4, 3), (65, 5, 4), (2, 1, 5), (70, 33, 12), (128, 64, 64), (250, 130, 17)])
def test_single_steps_give_the_bits_of_one_call(n, prec):
    import torch
    from paper_1804_01830_amd import binding as B
    w = W.random_stress(n, seed=73, d=(1.0, 1.5, 0.7))
    sig = torch.from_numpy(w["sigma"]).to("cuda", dtype=torch.float32 if prec == 32 else torch.float64).contiguous()
    us = []
    for parts in ((7,), (1,) * 7, (2, 0, 1, 3, 1)):
        r = B.Relax(n, w["d"], w["mu"], w["nu"], precision=prec)
        r.set_load(sig)
        for p in parts:
            r.iterate(p)
        us.append(r.displacement())
        torch.cuda.synchronize()
        r.close()
    print(f"[relax steps] {n} FP{prec}", flush=True)
    assert torch.equal(us[0], us[1]) and torch.equal(us[0], us[2])
