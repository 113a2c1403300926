"""The sources behind a traffic summary are those of every kernel of the passes, and
it takes the z launch that the library reported, whatever
its kernel (synthetic counter files, no GPU)."""
import csv
import os

from paper_1804_01830_amd import binding as B
from paper_1804_01830_amd import profiling as P

LINE = {"config": {"grid": [128, 128, 32], "workload": "sweep", "batch": 16},
        "plan_info": {"padded": [256, 256, 64], "tile_z": 16, "ez": 4, "z_groups": 1, "z_threads": 256,
                      "z_blocks": 4352},
        "roofline": {"kernel": "k_z_reg", "algorithmic_bytes_per_launch": 1000000}}


def _write(directory, counter, rows):
    os.makedirs(directory)
    with open(os.path.join(directory, "run_counter_collection.csv"), "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Workgroup_Size", "Grid_Size", "Counter_Name", "Counter_Value"])
        w.writerows([name, wg, grid, counter, val] for name, wg, grid, val in rows)


def test_traffic_of_the_register_form(tmp_path):
    z = "void dds::k_z_reg<64, 4, 6, true, 3, true>(dds::cplx<float> const*)"
    for counter, val in (("FETCH_SIZE", 400.0), ("WRITE_SIZE", 600.0)):
        _write(tmp_path / counter, counter, [(z, 256, 4352 * 256, val), (z, 128, 4352 * 128, 9e9),
                                             ("elementwise_kernel", 256, 1 << 20, 524288.0)])
    t = P.traffic(str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE"), LINE, 512)
    assert t["FETCH_SIZE"]["bytes"] == 400.0 * 1024 and t["WRITE_SIZE"]["bytes"] == 600.0 * 1024


def test_z_form_arguments_are_validated():
    out = B.ZLaunch()
    assert B.load().ddstress_plan_z_form(None, 1, out) == B.E_INVALID


def test_the_digest_covers_the_sources_of_every_pass():
    csrc = os.path.join(P.HERE, "csrc")
    # host code, the plan build, and kernels outside the five passes
    others = {"api.hip", "kernel_build.hip", "relax.hip", "stats.hip", "nye.hip"}
    assert {f"csrc/{f}" for f in os.listdir(csrc) if f.endswith((".hip", ".hpp")) and f not in others} == \
        set(P.DEVICE_SOURCES)
