"""Which kernels the library's host side launches for a call, and what it does
with graphs, tables and pinned memory while work is queued, without a GPU: the
host source linked against tests/host_route_driver.cpp, a stand-in of the HIP
runtime and of the kernel launchers whose clock runs as a scenario says."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = "/opt/rocm/bin/hipcc"

SCENARIOS = ["graph_in_flight", "tuning_between_batches", "no_steps_first",
             "form_reported_and_fixed", "tiles_that_are_resident",
             "cube_forms_by_estimate", "cubes_routed_one_by_one",
             "single_steps_time_no_field_form", "planes_routed_by_form",
             "staging_made_where_it_pays"]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("ROCm compiler not available")
    out = tmp_path_factory.mktemp("routes")
    csrc = os.path.join(ROOT, "paper_2306_10652_amd", "csrc")
    common = [HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17",
              "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
              "-I" + os.path.join(ROOT, "include"), "-I" + csrc, "-x", "hip", "-c"]
    objs = []
    procs = []
    for src in (os.path.join(csrc, "fuglbm_host.cpp"), os.path.join(HERE, "host_route_driver.cpp")):
        obj = str(out / (os.path.basename(src) + ".o"))
        objs.append(obj)
        procs.append(subprocess.Popen(common + [src, "-o", obj], stdout=subprocess.PIPE,
                                      stderr=subprocess.PIPE, text=True))
    for p in procs:
        _, err = p.communicate()
        assert p.returncode == 0, err[-3000:]
    exe = str(out / "routes")
    # linked without the HIP runtime: every call of it is the stand-in's
    r = subprocess.run(["/opt/rocm/llvm/bin/clang++"] + objs + ["-lpthread", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def test_scenarios_are_all_run(driver):
    r = subprocess.run([driver], capture_output=True, text=True, timeout=60)
    assert sorted(r.stdout.split()) == sorted(SCENARIOS)


@pytest.mark.parametrize("name", SCENARIOS)
def test_route(driver, name):
    r = subprocess.run([driver, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout[-2000:] + r.stderr[-2000:]
