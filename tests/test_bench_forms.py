"""What the benchmark reports of the form that its runs took, on the CPU: the
kernels' names and moved bytes follow the form that the library reports, the
stored counter summary of the field form's kernels was taken on their sources
as they are, and a step's traffic is put together from it."""
import json
import os
import sqlite3
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_field_counter_summary_matches_the_kernel_sources():
    import bench
    with open(bench.FIELD_PMC) as f:
        pm = json.load(f)
    assert pm["kernel_sha256_16"] == bench.kernel_hash(bench.FIELD_SRCS)
    b = {k: v["hbm_bytes_per_launch"] for k, v in pm["per_precision"]["fp64"].items()}
    assert bench.field_traffic("fp64", 1) == pytest.approx(b["eos"] + b["moments"] + b["last"])
    assert bench.field_traffic("fp64", 4) == pytest.approx(
        b["eos"] + 0.75 * b["step"] + 0.25 * (b["moments"] + b["last"]))
    # no less than the values that a long run cannot do without
    assert bench.field_traffic("fp64", 10 ** 9) > 59 * 8 * 1024 ** 2


def test_form_follows_the_library():
    import bench
    from paper_2306_10652_amd import capi
    sites, pop = 1024 ** 2, 2 * 10 * 1024 ** 2 * 72

    def result(code):
        return dict(csu_per_step=10 * sites, alg_bytes=pop, launch_ms=0.4, kernel=3,
                    achieved_gbs=pop / 0.4e-3 / 1e9, form_code=code)
    a, b = result(capi.FORM_POPULATIONS), result(capi.FORM_FIELDS)
    for r in (a, b):
        bench.field_form(r, 50)
    assert a["form"] == "populations every step" and "population_bytes" not in a
    assert b["population_bytes"] == pop and b["alg_bytes"] == 59 * 8 * sites + pop // 50
    assert bench.step_kernel(3, a["form_code"], "double") == "k_fused_d2q9_ws<10,double>"
    assert "k_field_step<10,double>" in bench.step_kernel(3, b["form_code"], "double")


def test_field_counter_summary_reads_rocprofv3_databases(tmp_path, capsys):
    import bench

    def db(name, counter, values):
        path = str(tmp_path / name)
        d = sqlite3.connect(path)
        d.execute("create table counters_collection "
                  "(dispatch_id int, kernel_name text, counter_name text, value real)")
        d.executemany("insert into counters_collection values (?,?,?,?)",
                      [(i, k, counter, v) for i, (k, v) in enumerate(values)])
        d.commit()
        d.close()
        return path

    def run(st, scale):
        k = "void fields::k_field_%s(FieldSim const*, int)"
        names = [k % n for n in ("moments<%s>" % st, "eos<10>", "step<10, %s, false>" % st,
                                 "step<10, %s, true>" % st)]
        trials = [(names[0], 9), (names[1], 9), (names[2], 9)]
        timed = [(names[0], 8), (names[1], 2), (names[2], 4), (names[1], 2), (names[3], 6)]
        return [(n, v * scale) for n, v in trials + timed]
    mib = 1 << 20
    copy = [("__amd_rocclr_copyBuffer", 512.0)]       # of 1024 KiB: the counter reads half
    paths = [db("f64", "FETCH_SIZE", run("double", 1)), db("w64", "WRITE_SIZE", run("double", 10)),
             db("f32", "FETCH_SIZE", run("float", 2)), db("w32", "WRITE_SIZE", run("float", 20)),
             db("cf", "FETCH_SIZE", copy), db("cw", "WRITE_SIZE", [(copy[0][0], 1024.0)])]
    out = str(tmp_path / "out.json")
    bench.pmc_field_summary(out, *paths, steps=2, copy_bytes=mib)
    capsys.readouterr()
    per = json.load(open(out))["per_precision"]
    got = {k: v["hbm_bytes_per_launch"] / 1024 for k, v in per["fp64"].items()}
    assert got == {"moments": 96, "eos": 24, "step": 48, "last": 72}     # 2 x fetch + write
    assert per["fp32"]["step"]["hbm_write_bytes_per_launch"] == 80 * 1024
